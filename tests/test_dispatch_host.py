"""paper_2505_19602_amd.routes against the rules that the library is built from: a host program around
csrc/common.h prints what they say for a grid of sizes."""
import os
import subprocess

import torch

from paper_2505_19602_amd import routes

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_19602_amd", "csrc")
UNITS = (1, 2, 9, 16, 31, 32, 40, 48, 63, 64, 80, 96, 111, 112, 127, 128, 129, 160, 161, 191, 192, 199, 200, 224, 225, 256, 257, 300,
         319, 320, 321, 383, 384, 512, 4000)
QUERIES = (1, 4, 16, 17, 32, 33, 64, 65, 100, 128, 129, 200, 256, 300, 448, 576, 1024, 1025, 2049, 4096)
KEYS = (1, 60, 117, 118, 256, 257, 320, 321, 326, 511, 512, 976, 977, 1023, 1024, 1280, 1281, 1400, 2000, 2001, 2999, 3000, 4096, 4097, 6500, 12288, 12289, 60000)
LENGTHS = (1, 2, 1535, 1536, 1537, 4096)   # cached rows: ranked in the launch that attends up to 1536
PROGRAM = """
#include <cstdio>
#include "common.h"
using namespace scalekv;
int main() {
  const int units[] = {%s}, queries[] = {%s}, keys[] = {%s};
  for (int u : units) for (int q : queries) for (int k : keys) {
    for (int dtype = 0; dtype < 2; ++dtype) for (int d = 64; d <= 128; d += 64) for (int w = 0; w < 4; ++w)
      printf("%%d ", small_tile_rows(dtype, d, u, q, k, (SmallWork)w));
    printf("%%d %%d\\n", (int)score_select_fits(1, 128, u, k), (int)asi_stream_pays(u, k, q));
  }
}
"""


def test_routes_are_the_rules_of_the_library(tmp_path):
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text(PROGRAM % tuple(", ".join(map(str, t)) for t in (UNITS, QUERIES, KEYS)))
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    lines = iter(subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=60).stdout.splitlines())
    for u in UNITS:
        for q in QUERIES:
            for k in KEYS:
                want = [routes.small_tile_rows(dtype, d, u, q, k, w) for dtype in (torch.float32, torch.bfloat16)
                        for d in (64, 128) for w in range(4)]
                want += [int(routes.ranks_in_one_launch(torch.bfloat16, u, k)),
                         int(routes.asi_streams(torch.bfloat16, u, k, q, 64))]
                assert [int(x) for x in next(lines).split()] == want, (u, q, k)
    assert next(lines, None) is None


# A step that keeps everything goes to the pipelined kernel where that has workgroups enough: a long cache in front of
# few units or few query tiles is walked by a few of them while the rest of the chip is idle, and a new cache that the
# last-level cache does not hold is copied at the pace of the compute units that have a unit in the last round.
def test_long_caches_that_are_kept_whole_go_where_the_chip_is_filled():
    kernel = lambda d, units, n, cached: routes.step_kernel(torch.bfloat16, d, units, n, cached, cached)
    for case in ((128, 128, 16, 5000), (128, 152, 5, 4200), (128, 272, 8, 3000), (128, 304, 5, 2500), (64, 272, 5, 5000),
                 (128, 16, 485, 4009), (128, 32, 254, 4473), (128, 64, 109, 2176), (64, 96, 37, 1812), (64, 128, 5, 800), (64, 20, 650, 101)):
        assert kernel(*case) == "small", case
    for case in ((128, 128, 10, 3000), (128, 168, 8, 4200), (128, 256, 8, 3000), (128, 288, 8, 1500), (128, 384, 8, 3000),
                 (64, 160, 8, 6000), (128, 48, 160, 800), (128, 40, 173, 221), (64, 128, 60, 800), (64, 168, 10, 800)):
        assert kernel(*case) == "pipelined", case


FORMS_PROGRAM = """
#include <cstdio>
#include "common.h"
using namespace scalekv;
int main() {
  const int units[] = {%s}, queries[] = {%s}, keys[] = {%s};
  for (int u : units) for (int q : queries) for (int k : keys)
    for (int d = 64; d <= 128; d += 64) {
      const PipeForm f = pipe_form(d, u, q, k);
      printf("%%s %%d %%d %%d %%d %%d\\n", f == PipeForm::kPlain ? "plain" : f == PipeForm::kWide ? "wide" : "split", pipe_rows(f),
             small_tile_rows(1, d, u, q, k, SmallWork::kRankedBefore), rows_go_past_caches(CacheWriter::kRanking, u, k, 2 * d),
             rows_go_past_caches(CacheWriter::kCompact, u, k, 2 * d), pipe_copies_cache(d, u, q, k));
    }
  const int lengths[] = {%s};
  for (int n : lengths) for (int keep : {0, 1, n - 1, n}) printf("%%d\\n", (int)step_work(keep, n));
}
"""


def test_forms_of_the_pipelined_kernel_are_the_rules_of_the_library(tmp_path):
    src, exe = tmp_path / "forms.hip", tmp_path / "forms"
    keys = KEYS + (319, 2047, 2048)
    src.write_text(FORMS_PROGRAM % tuple(", ".join(map(str, t)) for t in (UNITS, QUERIES, keys, LENGTHS)))
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    lines = iter(subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=60).stdout.splitlines())
    seen = set()
    for u in UNITS:
        for q in QUERIES:
            for k in keys:
                for d in (64, 128):
                    form = routes.pipe_form(d, u, q, k)
                    seen.add((d, form))
                    rows = routes.small_tile_rows(torch.bfloat16, d, u, q, k, routes.RANKED_BEFORE)
                    past = [int(routes.rows_go_past_caches(ranking, u, k, 2 * d)) for ranking in (True, False)]
                    copies = int(routes.pipe_copies_cache(d, u, q, k))
                    assert next(lines) == f"{form} {routes.pipe_rows(form)} {rows} {past[0]} {past[1]} {copies}", (u, q, k, d)
    for n in LENGTHS:
        for keep in (0, 1, n - 1, n):
            assert int(next(lines)) == routes.step_work(keep, n), (keep, n)
    assert next(lines, None) is None
    assert seen == {(64, "plain"), (64, "split"), (128, "plain"), (128, "wide"), (128, "split")}


SPREAD_PROGRAM = """
#include <cstdio>
#include "common.h"
using namespace scalekv;
int main() {
  const int units[] = {%s}, lengths[] = {%s};
  for (int u : units) for (int n : lengths) for (int d = 64; d <= 128; d += 64)
    printf("%%d %%d\\n", rank_spreads(d, u, n, true), rank_spreads(d, u, n, false));
  // a unit's workgroups share its rows and are at most the compute units
  for (int u : units) for (int n : lengths) {
    const int parts = select_parts(u, n);
    if (parts < 1 || (u <= 256 && u * parts > 256) || (parts > 1 && n / (parts - 1) < 64)) return 1;
  }
}
"""


def test_spread_ranking_is_the_rule_of_the_library(tmp_path):
    src, exe = tmp_path / "spread.hip", tmp_path / "spread"
    units = UNITS + (17, 24, 25, 33, 65, 97)
    lengths = LENGTHS + (799, 800, 999, 1000, 1299, 1300, 4097, 12288)
    src.write_text(SPREAD_PROGRAM % tuple(", ".join(map(str, t)) for t in (units, lengths)))
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    lines = iter(subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=60).stdout.splitlines())
    for u in units:
        for n in lengths:
            for d in (64, 128):
                assert next(lines) == f"{int(routes.rank_spreads(d, u, n, True))} {int(routes.rank_spreads(d, u, n, False))}", (u, n, d)
    assert next(lines, None) is None
