"""Which kernels a call takes, by its sizes: the dispatch rules of csrc/common.h, csrc/asi.hip and
csrc/api.hip in Python, for reports (bench.py prices each kernel against its own work) and for tests
that are written for one kernel.  tests/test_dispatch_host.py compares them with the C++ rules.
Output tensors that overlap inputs take other routes and are not covered."""
from __future__ import annotations

import torch

COMPUTE_UNITS = 256
ATTEND, APPEND, KEEP_ALL, RANKED, RANKED_BEFORE = range(5)   # enum class SmallWork
SHORT_LEN = 1536   # longest cache that is ranked in the launch that attends


def keep_all_is_pipelined(d: int, units: int, n_q: int, rows: int, n_wg: int, kv: int) -> bool:
    """Whether a step that keeps every row takes the pipelined kernel, which copies the tiles that pass."""
    n_pipe = units * -(-n_q // 128)
    if rows >= 64:
        return n_wg > 128 if d == 128 else n_wg > 192 and (n_wg >= 224 or n_pipe > 128 or kv >= 1024)
    if rows == 32 and n_pipe >= (96 if d == 128 else 112):
        return kv > 256
    if rows == 32:
        return 256 < kv <= 1280 and (units >= 96 or (d == 128 and units >= 32 and n_wg > 224))
    elements = units * kv * d
    if 4 * elements > 256 << 20:
        return 16 * units >= 10 * COMPUTE_UNITS * -(-units // COMPUTE_UNITS)
    idle = (units if d == 64 else n_wg) < 192
    return units >= 128 and elements >= (
        8_000_000 if idle else 5_000_000 if d == 64 else 2_000_000 if units >= 384 else 3_850_000)


def small_tile_rows(dtype: torch.dtype, d: int, units: int, n_q: int, kv: int, work: int) -> int:
    """Query rows per workgroup of the kernel for small work, 0 where it is not taken."""
    if dtype != torch.bfloat16:
        return 0
    for rows in (16, 32, 64, 128):
        n_wg = units * -(-n_q // rows)
        if n_wg <= COMPUTE_UNITS:
            break
    else:
        rows, n_wg = 256, units * -(-n_q // 128)
    if work == KEEP_ALL and keep_all_is_pipelined(d, units, n_q, 16 if rows > 128 else rows, n_wg, kv):
        return 0
    if rows > 128:
        return 16 if n_q <= 16 else 0
    if rows == 32 and work == ATTEND and kv <= 128:
        return 0
    if rows <= 32:
        return rows
    if rows == 128:
        return rows if work == RANKED and kv <= 320 else 0
    spare = n_wg <= COMPUTE_UNITS * 7 // 8
    pays = (work == RANKED and (d == 64 or n_q <= 1024)) or (work == RANKED_BEFORE and spare) or \
        work == KEEP_ALL or (work == APPEND and d == 64 and spare)
    return rows if pays else 0


def attend_kernel(dtype: torch.dtype, d: int, units: int, n_q: int, kv: int, work: int = ATTEND) -> str:
    """"f32", "small" or "pipelined"; work: ATTEND for scalekv_attend, APPEND for scalekv_step_append_first."""
    if dtype == torch.float32:
        return "f32"
    return "small" if small_tile_rows(dtype, d, units, n_q, kv, work) else "pipelined"


def pipe_form(d: int, units: int, n_q: int, kv: int) -> str:
    """The form of the pipelined kernel: "plain", "wide" or "split"."""
    wide, plain = units * -(-n_q // 256), units * -(-n_q // 128)
    if plain <= COMPUTE_UNITS:
        return "split" if kv >= 320 else "plain"
    if d != 128 or wide < COMPUTE_UNITS or kv < 2048:
        return "plain"
    rest = plain % (2 * COMPUTE_UNITS)
    plain_rounds = plain // (2 * COMPUTE_UNITS) * 100 + (0 if rest == 0 else 70 if rest <= COMPUTE_UNITS else 100)
    return "wide" if -(-wide // COMPUTE_UNITS) * 9600 <= plain_rounds * 100 else "plain"


def pipe_copies_cache(d: int, units: int, n_q: int, cached: int) -> bool:
    """Whether the pipelined kernel copies the rows of a cache that is kept whole; otherwise a launch before it does."""
    return pipe_form(d, units, n_q, cached + n_q) != "wide" or 2 * cached >= n_q


def pipe_rows(form: str) -> int:
    """Query rows per workgroup."""
    return 256 if form == "wide" else 128


def step_work(keep: int, cache_len: int) -> int:
    """What a step does besides the attention."""
    if 0 < keep < cache_len:
        return RANKED if cache_len <= SHORT_LEN else RANKED_BEFORE
    return KEEP_ALL if keep else APPEND


def rank_spreads(d: int, units: int, cache_len: int, small: bool) -> bool:
    """Whether several workgroups rank a unit, where ranks_in_one_launch(); small: its attention is in the kernel for
    small work."""
    if small and cache_len <= SHORT_LEN:
        return units <= (32 if cache_len >= 1000 else 16) and cache_len >= 800 if d == 128 else units <= 24 and cache_len >= 1300
    if small or units <= 64:
        return units <= 64 and cache_len >= (800 if d == 128 else 1300)
    return units <= (96 if cache_len <= 4096 else 128) and cache_len > SHORT_LEN if d == 128 else \
        units <= 96 and cache_len > 4096


def step_spreads(dtype: torch.dtype, d: int, units: int, n_cur: int, cache_len: int, budget: int) -> bool:
    """Whether scalekv_step ranks a unit by several workgroups."""
    keep = min(budget, cache_len)
    small = small_tile_rows(dtype, d, units, n_cur, keep + n_cur, step_work(keep, cache_len)) > 0
    return 0 < keep < cache_len and ranks_in_one_launch(dtype, units, cache_len) and rank_spreads(d, units, cache_len, small)


def step_kernel(dtype: torch.dtype, d: int, units: int, n_cur: int, cache_len: int, budget: int) -> str:
    """The same for the attention of scalekv_step; "small" appends in the same launch, and prunes unless the ranking has."""
    keep = min(budget, cache_len)
    work = step_work(keep, cache_len)
    if work == RANKED and step_spreads(dtype, d, units, n_cur, cache_len, budget) and \
            small_tile_rows(dtype, d, units, n_cur, keep + n_cur, work):
        work = RANKED_BEFORE
    return attend_kernel(dtype, d, units, n_cur, keep + n_cur, work)


def ranks_in_one_launch(dtype: torch.dtype, units: int, cache_len: int) -> bool:
    """Scores, selection and pruning of a unit by one workgroup (or inside the kernel for small work), unless
    rank_spreads()."""
    return dtype == torch.bfloat16 and cache_len <= 12288 and (units >= 64 or cache_len <= 4096)


def asi_streams(dtype: torch.dtype, units: int, length: int, n_samp: int, top_k: int) -> bool:
    """Selectivity without a workspace of logits."""
    if dtype != torch.bfloat16 or top_k > 256:
        return False
    rows, keys = min(n_samp, 32), units * length
    if min(units, 256) * rows >= (1024 if units >= 128 else 2048):
        return True
    return keys >= 160000 if rows == 32 else keys >= 220000 if rows >= 8 else keys >= 800000 and length >= 3000


def rows_go_past_caches(ranking: bool, units: int, rows: int, row_bytes: int) -> bool:
    """Whether the pruning stores its rows past the caches: by a ranking kernel or by compact_kernel."""
    return 2 * rows * units * row_bytes > (256_000_000 if ranking else 400_000_000)
