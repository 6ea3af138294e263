"""Sizes at which a kernel or a rule of its dispatch can go wrong: edges of tiles, remainders, the
smallest and largest of a range.  Everything is compared with the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_19602_amd as skv
import workloads as W
from paper_2505_19602_amd import routes
from parity_util import check_indices, check_output, units

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rand(key, shape, dtype, scale=1.0):
    return (W.normal_tensor(W.stream_key(4321, key), shape) * scale).to(dtype)


# 16 and 32 query rows per wave (by the workgroups of the fullest compute unit and the keys: (1, 40, 190, 241) and those
# behind it take 32 rows with head_dim 128, the last two with 64 too), 1, 2 and 4 waves sharing the keys, blocks that
# only some waves have, ragged blocks of 16 keys and of query rows, 16 rows with and without the LDS that keeps a third
# workgroup away (480 keys)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,n_q,kv_len", [
    (1, 2, 1, 1), (1, 2, 16, 15), (1, 3, 17, 16), (2, 2, 15, 17), (1, 2, 33, 48), (1, 2, 40, 63), (1, 2, 5, 65),
    (1, 1, 31, 129), (4, 48, 64, 33), (4, 48, 50, 80), (1, 100, 120, 20),
    (1, 40, 16, 511), (1, 40, 17, 512), (4, 80, 33, 513), (2, 64, 40, 527), (2, 64, 32, 97), (1, 40, 17, 479), (1, 40, 17, 480),
    (1, 40, 190, 241), (4, 64, 50, 263), (4, 64, 113, 240), (4, 64, 64, 529),
])
def test_attend_f32_edges(d, S, H, n_q, kv_len):
    print(f"attend f32 d={d} S={S} H={H} n_q={n_q} kv_len={kv_len}", flush=True)
    shape = skv.Shape(S, H, d, torch.float32)
    q, k, v = (_rand(1 + i, (S, H, n, d), torch.float32, 1.3) for i, n in enumerate((n_q, kv_len + 3, kv_len + 3)))
    k[:, :, kv_len:] = float("nan"); v[:, :, kv_len:] = float("nan")
    out = torch.full((S, H, n_q + 1, d), 7.0, device=DEV)
    flat = out.reshape(-1)[: S * H * n_q * d].view(S, H, n_q, d)      # rows behind the output must stay
    skv.attend(shape, q.to(DEV), k.to(DEV), v.to(DEV), kv_len, flat)
    torch.cuda.synchronize()
    assert torch.all(out.reshape(-1)[S * H * n_q * d:] == 7.0)
    pick = sorted({0, S * H // 2, S * H - 1})
    ref = oracle.attend(units(q)[pick], units(k)[pick][:, :kv_len], units(v)[pick][:, :kv_len])
    check_output(units(flat)[pick], ref, torch.float32, "attend f32")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,n_win", [(1, 1), (63, 3), (64, 16), (65, 4), (255, 5), (257, 16), (700, 13)])
def test_score_f32_edges(d, L, n_win):
    S, H = 1, 3
    print(f"score f32 d={d} L={L} n_win={n_win}", flush=True)
    shape = skv.Shape(S, H, d, torch.float32)
    qw, k = _rand(5, (S, H, n_win, d), torch.float32, 1.5), _rand(6, (S, H, L + 2, d), torch.float32, 1.5)
    ls = torch.full((S, H, L), float("nan"), device=DEV)
    ws = torch.empty(skv.workspace_bytes(shape, L, 16), dtype=torch.uint8, device=DEV)
    skv.score(shape, qw.to(DEV), k.to(DEV), L, ls, ws)
    torch.cuda.synchronize()
    _, ref = oracle.score(units(qw), units(k)[:, :L])
    assert np.abs(ls.cpu().numpy().reshape(S * H, L).astype(np.float64) - ref).max() < 2e-4


# tiles of 16 keys, waves of 64 and chunks of 256, channels of very different sizes.  A logit is a sum of d products: its
# error is at most d 2^-24 of the sum of their magnitudes, the row normaliser's as much; exp, log: a few 2^-24 of about 10.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,n_win", [(15, 16), (16, 1), (17, 15), (192, 9), (193, 16), (256, 2), (513, 16)])
def test_score_f32_tiles(d, L, n_win):
    S, H = 2, 2
    print(f"score f32 tiles d={d} L={L} n_win={n_win}", flush=True)
    shape = skv.Shape(S, H, d, torch.float32)
    qw, k = _rand(7, (S, H, n_win, d), torch.float32, 1.5), _rand(8, (S, H, L + 1, d), torch.float32, 1.5)
    qw[:, :, :, ::3] *= 2.0 ** 10
    k[:, :, :, ::3] *= 2.0 ** -10
    k[:, :, L:] = float("nan")
    ls = torch.full((S, H, L), float("nan"), device=DEV)
    ws = torch.empty(skv.workspace_bytes(shape, L, 16), dtype=torch.uint8, device=DEV)
    skv.score(shape, qw.to(DEV), k.to(DEV), L, ls, ws)
    torch.cuda.synchronize()
    _, ref = oracle.score(units(qw), units(k)[:, :L])
    bound = (d * 2.0 ** -24 * (qw.abs() @ k[:, :, :L].abs().transpose(2, 3)).max() / d ** 0.5).item()
    assert np.abs(ls.cpu().numpy().reshape(S * H, L).astype(np.float64) - ref).max() < 2 * bound + 2e-5


def _step_against_oracle(S, H, d, L, budget, n_cur, n_win, pick, seed, dup=1, idx_of=None):
    """One step; units `pick` followed by the oracle.  dup > 1: cached rows repeat in runs of that length (ties).
    idx_of: the indices of the same step; it is then called without an index list.  Returns its outputs and indices."""
    dtype = torch.bfloat16
    shape = skv.Shape(S, H, d, dtype)
    keep = min(budget, L)
    mk = lambda i, n, scale=1.0: _rand(100 * seed + i, (S, H, n, d), dtype, scale)
    q, kc, vc, vs = mk(0, n_cur, 1.5), mk(1, n_cur), mk(2, n_cur), mk(3, L + 2)
    ks = mk(4, (L + 2 + dup - 1) // dup, 1.5).repeat_interleave(dup, 2)[:, :, : L + 2].contiguous()
    ks[:, :, L:] = float("nan"); vs[:, :, L:] = float("nan")
    win = list(range(n_cur - n_win, n_cur))
    cap = keep + n_cur + 2
    kd = torch.full((S, H, cap, d), 7.0, dtype=dtype, device=DEV); vd = torch.full_like(kd, 7.0)
    out = torch.full((S, H, n_cur, d), float("nan"), dtype=dtype, device=DEV)
    idx = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV) if idx_of is None else None
    ws = torch.empty(skv.workspace_bytes(shape, max(L, 1), n_cur), dtype=torch.uint8, device=DEV)
    assert skv.step(shape, q.to(DEV), kc.to(DEV), vc.to(DEV), win, ks.to(DEV), vs.to(DEV), L, budget, kd, vd, out, idx,
                    ws) == keep + n_cur
    torch.cuda.synchronize()
    for t in (kd, vd):
        assert torch.all(t[:, :, keep + n_cur:] == 7.0)
    sub = lambda t: units(t)[pick]
    kpart, vpart = sub(ks)[:, :L], sub(vs)[:, :L]
    if keep and keep < L:
        _, ls = oracle.score(sub(q)[:, win], kpart)
        own = oracle.select(ls, budget)
    else:
        ls, own = np.zeros((len(pick), L)), np.tile(np.arange(keep), (len(pick), 1))
    idx = idx if idx_of is None else idx_of
    got = idx.cpu().numpy().reshape(S * H, keep)[pick]
    for u in range(len(pick)):
        if dup == 1:
            check_indices(got[u], ls[u], keep, own[u])
        else:      # equal rows have equal scores: of a run that is cut, the lower rows are kept
            assert np.array_equal(got[u], own[u])
    ref = oracle.step(sub(q), sub(kc), sub(vc), win, kpart, vpart, budget, force_idx=got)
    assert np.array_equal(sub(kd)[:, : keep + n_cur].double().numpy(), ref["k_dst"])
    assert np.array_equal(sub(vd)[:, : keep + n_cur].double().numpy(), ref["v_dst"])
    check_output(sub(out), ref["out"], dtype, "step")
    return kd, vd, out, idx


# Small steps: groups of 32 keys, rounds of 512 keys, the longest cache ranked in LDS and the first beyond it (with few
# units, from 800 rows on, head_dim 64 from 1300, ranked by several workgroups to a unit; one launch at those lengths:
# test_one_launch_ranking_of_longer_caches); 16-query blocks, several blocks per workgroup (many units), ties.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,L,budget,n_cur,n_win,dup", [
    (1, 2, 2, 1, 1, 1, 1), (1, 3, 31, 30, 15, 15, 1), (1, 2, 33, 1, 16, 16, 1), (2, 2, 64, 32, 17, 3, 1),
    (1, 2, 511, 100, 40, 16, 1), (1, 2, 513, 512, 33, 16, 1), (1, 2, 1025, 77, 64, 16, 1), (1, 2, 1535, 400, 128, 16, 1),
    (1, 2, 1536, 1535, 20, 16, 1), (1, 2, 1537, 500, 20, 16, 1), (4, 80, 200, 50, 128, 16, 1), (3, 100, 90, 20, 50, 16, 1),
    (2, 140, 300, 60, 30, 16, 1), (1, 2, 300, 101, 20, 16, 5), (1, 2, 1200, 333, 36, 16, 7), (1, 1, 40, 13, 5, 5, 40),
    (1, 2, 50, 50, 20, 16, 1), (1, 2, 40, 0, 20, 16, 1), (40, 20, 60, 60, 100, 16, 1),
])
def test_small_step_edges(d, S, H, L, budget, n_cur, n_win, dup):
    print(f"small step d={d} S={S} H={H} L={L} budget={budget} n_cur={n_cur} n_win={n_win} dup={dup}", flush=True)
    pick = sorted({0, S * H // 2, S * H - 1})
    kept = _step_against_oracle(S, H, d, L, budget, n_cur, n_win, pick, 1, dup)
    # the same step without an index list to write: what is kept, and everything else, must not change
    for a, b in zip(kept, _step_against_oracle(S, H, d, L, budget, n_cur, n_win, pick, 1, dup, idx_of=kept[3])):
        assert torch.equal(a, b)


# The kernel for small work where the kept rows are known before it: one chunk of 32 keys to each of its eight (64 query
# rows: four) waves at most, and the first length with which one has two; some without any; rows kept by a ranking (few
# of many, through the index list) and whole caches; 16, 32 and 64 query rows to a workgroup
@pytest.mark.parametrize("d,S,H,L,budget,n_cur", [
    (d, 1, 3, L, budget, n) for d in (64, 128) for L, budget, n in (
        (1700, 235, 20), (1700, 236, 20), (1700, 237, 20), (2000, 1, 1), (1, 1, 1), (31, 31, 1), (32, 32, 1), (235, 235, 20),
        (236, 236, 20), (237, 237, 20), (500, 500, 17))
] + [(128, 2, 50, 216, 216, 40), (128, 2, 20, 217, 217, 100), (64, 2, 50, 215, 215, 40), (64, 2, 48, 57, 57, 70),
     (64, 2, 48, 58, 58, 70), (64, 2, 48, 59, 59, 70)])
def test_one_chunk_to_a_wave(d, S, H, L, budget, n_cur):
    print(f"one chunk to a wave d={d} S={S} H={H} L={L} budget={budget} n_cur={n_cur}", flush=True)
    assert routes.step_kernel(torch.bfloat16, d, S * H, n_cur, L, budget) == "small"
    _step_against_oracle(S, H, d, L, budget, n_cur, min(16, n_cur), sorted({0, S * H // 2, S * H - 1}), 21)


# Caches of 800 to 1536 rows that are ranked in the launch that attends: more units than rank_spreads() takes.
@pytest.mark.parametrize("d,S,H,L,budget,n_cur,n_win,dup", [
    (128, 1, 17, 800, 60, 20, 16, 1), (128, 1, 32, 999, 300, 16, 5, 1), (128, 3, 11, 1025, 77, 64, 16, 1), (128, 1, 33, 1200, 333, 36, 16, 7),
    (128, 3, 11, 1535, 400, 128, 16, 1), (128, 1, 33, 1536, 1535, 20, 16, 1), (128, 3, 11, 1536, 700, 420, 16, 1),
    (64, 1, 25, 1300, 60, 20, 16, 1), (64, 5, 5, 1535, 400, 128, 16, 1), (64, 5, 5, 1536, 1535, 20, 16, 1),
])
def test_one_launch_ranking_of_longer_caches(d, S, H, L, budget, n_cur, n_win, dup):
    print(f"one launch d={d} S={S} H={H} L={L} budget={budget} n_cur={n_cur} n_win={n_win} dup={dup}", flush=True)
    assert routes.step_kernel(torch.bfloat16, d, S * H, n_cur, L, budget) == "small"
    assert not routes.step_spreads(torch.bfloat16, d, S * H, n_cur, L, budget)
    _step_against_oracle(S, H, d, L, budget, n_cur, n_win, sorted({0, S * H // 2, S * H - 1}), 31, dup)


# Short caches are selected by counting, four lanes or two to a row (512 threads: up to 128 and 256 rows; the ranking
# kernel with 1024: 256): shares of four keys and their remainders, the first length beyond; runs of equal rows that
# the border cuts or not, and rows that are all equal, which the search decides.
@pytest.mark.parametrize("S,H,n_cur", [(1, 3, 20), (4, 50, 300)])
@pytest.mark.parametrize("L,budget", [(5, 2), (16, 15), (17, 8), (127, 60), (128, 1), (129, 128), (255, 90), (256, 255),
                                      (257, 30)])
@pytest.mark.parametrize("dup", [1, 3, 1000])
def test_selection_of_short_caches(S, H, n_cur, L, budget, dup):
    print(f"short selection {S}x{H} L={L} budget={budget} n_cur={n_cur} dup={dup}", flush=True)
    _step_against_oracle(S, H, 64, L, budget, n_cur, 16, sorted({0, S * H - 1}), 11, dup)


# The ranking of a unit spread over workgroups against a workgroup per unit: a step of many units takes the second, a
# step of the first `few` of them the first, and both keep the same rows, bit for bit, and copy them.  Lengths around
# groups of 32, 128 and 256 keys and rounds of 16 groups, rows per thread of the selection, shares of the pruning
# (1 to 85 workgroups), tied rows; with the attention that appends and the one that does not.
@pytest.mark.parametrize("d,few,n_cur,L,budget,n_win,dup", [
    (128, 3, 20, 800, 1, 1, 1), (128, 3, 300, 801, 800, 16, 1), (128, 32, 256, 1023, 77, 7, 1), (128, 1, 16, 1024, 500, 16, 3),
    (128, 64, 300, 1025, 256, 16, 1), (128, 2, 40, 1535, 129, 9, 1), (128, 64, 300, 1536, 1535, 16, 5), (128, 96, 300, 1537, 300, 16, 1),
    (128, 3, 20, 2047, 40, 16, 1), (128, 64, 20, 2049, 900, 4, 1), (128, 5, 300, 4096, 1000, 16, 7), (128, 64, 130, 4097, 700, 16, 1),
    (128, 96, 130, 8191, 600, 16, 1), (128, 64, 20, 12288, 5000, 16, 1),
    (64, 3, 20, 1300, 64, 16, 1), (64, 64, 1300, 1337, 65, 3, 2), (64, 1, 40, 1536, 1000, 16, 1), (64, 64, 40, 2048, 63, 16, 1),
    (64, 96, 300, 5000, 1250, 16, 1),
])
def test_spread_ranking_keeps_the_same_rows(d, few, n_cur, L, budget, n_win, dup):
    print(f"spread ranking d={d} few={few} n_cur={n_cur} L={L} budget={budget} n_win={n_win} dup={dup}", flush=True)
    many, dtype = 130, torch.bfloat16
    assert routes.step_spreads(dtype, d, few, n_cur, L, budget) and not routes.step_spreads(dtype, d, many, n_cur, L, budget)
    gen = torch.Generator(device=DEV).manual_seed(L + few)
    mk = lambda n, scale=1.0: (torch.randn(1, many, n, d, device=DEV, generator=gen) * scale).to(dtype)
    q, kc, vc, vs = mk(n_cur, 1.5), mk(n_cur), mk(n_cur), mk(L)
    ks = mk((L + dup - 1) // dup, 1.5).repeat_interleave(dup, 2)[:, :, :L].contiguous()
    win = list(range(n_cur - n_win, n_cur))

    def run(units):
        part = lambda t: t[:, :units].clone()
        shape = skv.Shape(1, units, d, dtype)
        kd = torch.full((1, units, budget + n_cur + 1, d), 7.0, dtype=dtype, device=DEV); vd = torch.full_like(kd, 7.0)
        out, idx = torch.zeros(1, units, n_cur, d, dtype=dtype, device=DEV), torch.full((1, units, budget), -1, dtype=torch.int32, device=DEV)
        ws = torch.empty(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
        skv.step(shape, part(q), part(kc), part(vc), win, part(ks), part(vs), L, budget, kd, vd, out, idx, ws)
        # the literal order: forced window rows, pooled scores, `L` rows in all
        k_all, v_all = part(ks), part(vs)
        keep = n_win + min(budget, L - n_win - 1)
        kn = torch.full((1, units, keep + 1, d), 7.0, dtype=dtype, device=DEV); vn = torch.full_like(kn, 7.0)
        idx2 = torch.full((1, units, keep), -1, dtype=torch.int32, device=DEV)
        skv.step_append_first(shape, part(q), part(kc), part(vc), win, 3, k_all, v_all, L - n_cur, keep - n_win, kn, vn, out.clone(),
                              idx2, ws)
        torch.cuda.synchronize()
        return idx, kd, vd, idx2, kn, vn

    for a, b in zip(run(few), run(many)):
        assert torch.equal(a, b[:, :few])


# fp32: selection and pruning in one launch (up to 256 units, one or several workgroups each) against two (257), rows
# per thread of the selection, log-scores formed in it (up to 2048 rows) or before, the longest for which it holds
@pytest.mark.parametrize("d,few,L,budget,n_cur", [
    (128, 256, 2, 1, 20), (64, 256, 300, 299, 17), (128, 3, 1024, 65, 20), (64, 1, 1025, 1000, 20), (128, 100, 2048, 128, 30),
    (128, 7, 2049, 64, 20), (64, 130, 4097, 129, 20), (64, 20, 8193, 2000, 20), (64, 2, 12288, 300, 20), (64, 2, 12289, 300, 20),
])
def test_selection_that_prunes_f32(d, few, L, budget, n_cur):
    print(f"selection and pruning f32 d={d} few={few} L={L} budget={budget} n_cur={n_cur}", flush=True)
    many, dtype = 257, torch.float32
    gen = torch.Generator(device=DEV).manual_seed(L + few)
    mk = lambda n: torch.randn(1, many, n, d, device=DEV, generator=gen)
    q, kc, vc, ks, vs = mk(n_cur), mk(n_cur), mk(n_cur), mk(L), mk(L)
    n_win = min(16, n_cur)
    win = list(range(n_cur - n_win, n_cur))

    def run(units):
        part = lambda t: t[:, :units].clone()
        shape = skv.Shape(1, units, d, dtype)
        kd = torch.full((1, units, budget + n_cur + 1, d), 7.0, device=DEV); vd = torch.full_like(kd, 7.0)
        out, idx = torch.zeros(1, units, n_cur, d, device=DEV), torch.full((1, units, budget), -1, dtype=torch.int32, device=DEV)
        ws = torch.empty(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
        skv.step(shape, part(q), part(kc), part(vc), win, part(ks), part(vs), L, budget, kd, vd, out, idx, ws)
        torch.cuda.synchronize()
        return idx, kd, vd

    got, want = run(few), run(many)
    for a, b in zip(got, want):
        assert torch.equal(a, b[:, :few])
    rows = got[0].long().unsqueeze(-1).expand(-1, -1, -1, d)
    for dst, src, cur in ((got[1], ks, kc), (got[2], vs, vc)):
        assert torch.equal(dst[:, :, :budget], src[:, :few].gather(2, rows))
        assert torch.equal(dst[:, :, budget:-1], cur[:, :few]) and torch.all(dst[:, :, -1] == 7.0)


# four lanes to a row up to 128 rows, two up to 256 (1024 threads, as with the 150 units x 300 queries: 256 and 256),
# then one; windows that leave some of those lanes without a row of their own
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,n_cur", [(1, 3, 20), (3, 50, 300)])
@pytest.mark.parametrize("L,budget", [(2, 1), (33, 9), (128, 50), (129, 50), (256, 90), (257, 90), (520, 100)])
@pytest.mark.parametrize("n_win", [1, 4, 7, 9, 15])
def test_window_sizes_of_short_rankings(d, S, H, n_cur, L, budget, n_win):
    print(f"window of a short ranking d={d} S={S} H={H} n_cur={n_cur} L={L} budget={budget} n_win={n_win}", flush=True)
    _step_against_oracle(S, H, d, L, budget, n_cur, n_win, sorted({0, S * H - 1}), 71 + L + n_win)


# Streamed selectivity: rounds of 512 keys, lists that overflow and are cut (keys in ascending order of
# their scores), ties at the threshold, several parts per unit, one and two blocks of 16 rows, history
# within a round, K' at its limits and beyond (the route through the logits)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,n_samp,hist,cur,top_k,kind", [
    (1, 2, 1, 1, 1, 1, "normal"), (1, 2, 16, 0, 40, 64, "normal"), (1, 2, 17, 511, 1, 64, "normal"),
    (1, 2, 33, 513, 31, 200, "normal"), (1, 2, 16, 2000, 100, 256, "rising"), (1, 2, 5, 3000, 500, 64, "rising"),
    (1, 2, 20, 1025, 0, 16, "ties"), (2, 2, 16, 1500, 600, 1500, "normal"), (1, 2, 16, 900, 50, 257, "normal"),
    (1, 2, 16, 5000, 30, 255, "ties"), (3, 50, 8, 1100, 70, 0, "normal"), (9, 16, 32, 700, 400, 100, "rising"),
    # (few units and few keys take the route through the logits: the same edges with enough of them)
    (16, 16, 4, 1, 1, 1, "normal"), (8, 16, 16, 0, 40, 64, "normal"), (8, 16, 17, 511, 1, 64, "normal"),
    (8, 16, 33, 513, 31, 200, "normal"), (8, 16, 16, 2000, 100, 256, "rising"), (16, 16, 5, 3000, 500, 64, "rising"),
    (8, 16, 20, 1025, 0, 16, "ties"), (8, 16, 16, 200, 50, 256, "normal"), (8, 16, 16, 5000, 30, 255, "ties"),
    (16, 16, 1, 3100, 400, 64, "rising"), (1, 16, 32, 9500, 600, 64, "rising"), (1, 2, 40, 80500, 10, 200, "rising"),
])
def test_asi_edges(d, S, H, n_samp, hist, cur, top_k, kind):
    print(f"asi d={d} S={S} H={H} n_samp={n_samp} hist={hist} cur={cur} top_k={top_k} {kind}", flush=True)
    dtype, n = torch.bfloat16, hist + cur
    assert routes.asi_streams(dtype, S * H, n, n_samp, top_k) == (S * H > 10 or n > 50000)
    shape = skv.Shape(S, H, d, dtype)
    q = _rand(7, (S, H, n_samp, d), dtype, 1.5).to(DEV)
    k = W.normal_tensor(W.stream_key(4321, 8), (S, H, n, d), DEV)
    if kind == "rising":       # scores of every query grow along the cache
        q = (q.float() * 0.2 + 1.0).to(dtype)
        k = k * 0.1 + torch.linspace(-0.5, 0.5, n).to(DEV)[None, None, :, None]
    elif kind == "ties":
        k = k.repeat_interleave(9, 2)[:, :, :n]
    k = k.to(dtype)
    terms = torch.full((S, H, n_samp, 2), float("nan"), device=DEV)
    mean = torch.empty(3, device=DEV)
    ws = torch.empty(skv.workspace_bytes(shape, n, n_samp), dtype=torch.uint8, device=DEV)
    skv.asi(shape, q.to(DEV), k.to(DEV), hist, cur, top_k, terms, mean, ws)
    again = torch.empty_like(terms)
    skv.asi(shape, q.to(DEV), k.to(DEV), hist, cur, top_k, again, mean, ws)
    torch.cuda.synchronize()
    assert torch.equal(terms, again)
    pick = sorted({0, S * H - 1})
    ref = np.stack(oracle.asi_terms(units(q)[pick], units(k)[pick], hist, top_k), -1)
    got = terms.cpu().numpy().reshape(S * H, n_samp, 2)[pick].astype(np.float64)
    assert np.abs(got - ref).max() < 2e-5


# Ranking in front of the pipelined attention (150 queries of 300 units, or 2049 queries): caches ranked in
# LDS, in registers (rounds of 512 keys, two at a time) and beyond, with and without a unit per compute
# unit; then the route for few units with long caches
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,L,budget,n_cur,dup", [
    (1, 10, 1537, 3, 2049, 1), (1, 9, 2047, 2046, 2049, 1), (1, 9, 2049, 700, 2049, 6), (1, 9, 3585, 900, 2049, 1),
    (1, 9, 4096, 4095, 2049, 1), (1, 9, 4095, 1, 2049, 4), (4, 40, 1600, 200, 300, 1), (4, 75, 700, 90, 150, 1),
    (4, 75, 1700, 90, 150, 1), (1, 2, 4097, 800, 20, 1), (1, 2, 6400, 1000, 20, 3), (4, 16, 4100, 300, 900, 1),
])
def test_rank_edges(d, S, H, L, budget, n_cur, dup):
    print(f"rank d={d} S={S} H={H} L={L} budget={budget} n_cur={n_cur} dup={dup}", flush=True)
    _step_against_oracle(S, H, d, L, budget, n_cur, 16, sorted({0, S * H - 1}), 2, dup)


# Forced rows beside the search: with the largest and the smallest scores of the unit, next to the threshold, among
# equal scores, all that is kept; units of 1, 2, 4, 8 and 12 rows a thread, and the route that leaves LDS
@pytest.mark.parametrize("L", [17, 1024, 1025, 2049, 4097, 8192, 8193, 12288, 12289])
@pytest.mark.parametrize("kind", ["spread", "close", "equal"])
@pytest.mark.parametrize("pool_w", [1, 5])
def test_select_with_forced_rows_edges(L, kind, pool_w):
    S, H = 1, 3
    print(f"forced rows L={L} {kind} pool_w={pool_w}", flush=True)
    shape = skv.Shape(S, H, 64, torch.bfloat16)
    ls = W.normal_tensor(W.stream_key(4321, 120 + L), (S, H, L)) * {"spread": 4.0, "close": 0.01, "equal": 0.0}[kind] - 5.0
    order = torch.argsort(ls[0, 0])
    for budget in sorted({0, 1, min(L // 3, L - 17), L - 17} - {-1}):
        for forced in ([int(order[0])], [int(order[-1]), int(order[0])], sorted({0, L - 1, *order[-max(1, budget):][:14].tolist()})):
            if len(forced) + budget >= L:
                continue
            keep = len(forced) + budget
            idx = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV)
            assert skv.select_window(shape, ls.to(DEV), L, budget, forced, pool_w, idx) == keep
            torch.cuda.synchronize()
            got = idx.cpu().numpy().reshape(S * H, keep)
            pooled = oracle.pool_log(ls.double().numpy().reshape(S * H, L), pool_w)
            if pool_w == 1:
                assert np.array_equal(got, oracle.select_forced(pooled, budget, forced))
                continue
            for u in range(S * H):
                rest = np.setdiff1d(got[u], forced)
                assert set(forced) <= set(got[u].tolist()) and np.all(np.diff(got[u]) > 0) and len(rest) == budget
                if budget:   # nothing left out lies above what was taken: both within 4 ulp of 32 (2^-19 each) of the exact
                    out = np.setdiff1d(np.arange(L), got[u])
                    assert pooled[u][rest].min() >= pooled[u][out].max() - 8 * 2.0 ** -19


# out in the place of q: the workgroups of a unit must not read the window after a neighbour has written (12 units, 1536
# rows: ranked by launches of their own in any case)
@pytest.mark.parametrize("d,L,budget,n_cur,H", [(64, 700, 90, 200, 12), (128, 1536, 300, 128, 12), (128, 1536, 300, 128, 40),
                                                (128, 90, 20, 16, 12)])
def test_small_step_writes_over_its_queries(d, L, budget, n_cur, H):
    S, dtype = 1, torch.bfloat16
    print(f"out over q d={d} H={H} L={L} budget={budget} n_cur={n_cur}", flush=True)
    assert routes.step_kernel(dtype, d, H, n_cur, L, budget) == "small"
    assert routes.step_spreads(dtype, d, H, n_cur, L, budget) == ((H, L) == (12, 1536))
    shape = skv.Shape(S, H, d, dtype)
    q, kc, vc, ks, vs = (_rand(60 + i, (S, H, n, d), dtype, 1.3).to(DEV) for i, n in enumerate((n_cur,) * 3 + (L,) * 2))
    ws = torch.empty(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
    results = []
    for over in (False, True):
        out = q if over else torch.empty_like(q)
        kd = torch.empty(S, H, budget + n_cur, d, dtype=dtype, device=DEV); vd = torch.empty_like(kd)
        skv.step(shape, q, kc, vc, list(range(n_cur - 16, n_cur)), ks, vs, L, budget, kd, vd, out, None, ws)
        torch.cuda.synchronize()
        results.append((out, kd, vd))
    for plain, over in zip(*results):
        assert torch.equal(plain, over)


# out on top of the map's keys or values, or of the source cache: all of them are read before it is stored
@pytest.mark.parametrize("d,H,L,budget,n_cur", [(64, 12, 700, 90, 200), (128, 12, 90, 20, 16), (128, 12, 40, 40, 100),
                                                (128, 6, 1600, 200, 120), (64, 40, 300, 60, 1100)])
@pytest.mark.parametrize("over", ["k_cur", "v_cur", "k_src", "v_src"])
def test_step_writes_over_its_inputs(over, d, H, L, budget, n_cur):
    dtype = torch.bfloat16
    print(f"out over {over} d={d} H={H} L={L} budget={budget} n_cur={n_cur}", flush=True)
    shape = skv.Shape(1, H, d, dtype)
    q, kc, vc = (_rand(80 + i, (1, H, n_cur, d), dtype, 1.3).to(DEV) for i in range(3))
    ks, vs = (_rand(83 + i, (1, H, max(L, n_cur), d), dtype, 1.3).to(DEV) for i in range(2))
    ws = torch.empty(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
    win = list(range(n_cur - 16, n_cur))
    in_q, in_kc, in_vc, in_ks, in_vs = (units(t).clone() for t in (q, kc, vc, ks[:, :, :L], vs[:, :, :L]))
    if over in ("k_src", "v_src"):
        out = (ks if over == "k_src" else vs).view(-1)[:q.numel()].view_as(q)
    else:
        out = kc if over == "k_cur" else vc
    kd = torch.empty(1, H, budget + n_cur, d, dtype=dtype, device=DEV); vd = torch.empty_like(kd)
    idx = torch.empty(1, H, budget, dtype=torch.int32, device=DEV)
    skv.step(shape, q, kc, vc, win, ks, vs, L, budget, kd, vd, out, idx, ws)
    torch.cuda.synchronize()
    kept = idx.cpu()[0]
    for u in range(H):      # every unit's rows; whose selection and output are right: the first, a middle and the last
        rows = kept[u].long()
        assert torch.equal(kd[0, u].cpu(), torch.cat([in_ks[u][rows], in_kc[u]]))
        assert torch.equal(vd[0, u].cpu(), torch.cat([in_vs[u][rows], in_vc[u]]))
    pick = [0, H // 2, H - 1]
    if budget < L:
        _, ls = oracle.score(in_q[pick][:, win], in_ks[pick])
        own = oracle.select(ls, budget)
        for i, u in enumerate(pick):
            check_indices(kept[u].numpy(), ls[i], budget, own[i])
    ref = oracle.step(in_q[pick], in_kc[pick], in_vc[pick], win, in_ks[pick], in_vs[pick], budget,
                      force_idx=kept[pick].numpy())
    check_output(units(out)[pick], ref["out"], dtype, "step")


# keys whose logits are all -inf have weight zero, also where one wave meets nothing else
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,n_q", [(64, 20), (128, 33)])
def test_attend_over_keys_of_weight_zero(dtype, d, n_q):
    S, H, kv = 1, 2, 200
    print(f"weight zero d={d} n_q={n_q} {dtype}", flush=True)
    shape = skv.Shape(S, H, d, dtype)
    q, k, v = (_rand(70 + i, (S, H, n, d), dtype) for i, n in enumerate((n_q, kv, kv)))
    q[..., 0] = 1.0
    keep = torch.ones(kv, dtype=torch.bool)
    keep[16:32] = False; keep[64:96] = False
    k[:, :, ~keep, 0] = float("-inf")
    out = torch.empty(S, H, n_q, d, dtype=dtype, device=DEV)
    skv.attend(shape, q.to(DEV), k.to(DEV), v.to(DEV), kv, out)
    torch.cuda.synchronize()
    ref = oracle.attend(units(q), units(k)[:, keep], units(v)[:, keep])
    check_output(units(out), ref, dtype, "attend")


# the same where the logits are scaled by one and more (queries and keys that are normalised): 16 and 32 query rows
# per workgroup, a wave that meets nothing but such keys
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("sm_scale", [0.7, 1.0, 8.0])
@pytest.mark.parametrize("d,H,n_q", [(64, 2, 20), (128, 2, 33), (64, 20, 200), (128, 20, 200)])
def test_attend_over_keys_of_weight_zero_at_other_scales(dtype, sm_scale, d, H, n_q):
    kv = 200
    print(f"weight zero d={d} H={H} n_q={n_q} sm_scale={sm_scale} {dtype}", flush=True)
    shape = skv.Shape(1, H, d, dtype, sm_scale)
    q, k, v = (_rand(90 + i, (1, H, n, d), dtype) for i, n in enumerate((n_q, kv, kv)))
    q = (q.float() / (sm_scale * d ** 0.5)).to(dtype)
    q[..., 0] = 0.125
    keep = torch.ones(kv, dtype=torch.bool)
    keep[16:32] = False; keep[64:96] = False
    k[:, :, ~keep, 0] = float("-inf")
    out = torch.empty(1, H, n_q, d, dtype=dtype, device=DEV)
    skv.attend(shape, q.to(DEV), k.to(DEV), v.to(DEV), kv, out)
    torch.cuda.synchronize()
    ref = oracle.attend(units(q), units(k)[:, keep], units(v)[:, keep], sm_scale)
    check_output(units(out), ref, dtype, "attend")


# the same in the pipelined kernel (more than 256 units): a first block, a first tile and a second tile of such keys;
# then as cache and map of a step, where the map's keys are a second segment
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q", [20, 150])
@pytest.mark.parametrize("lo,hi", [(0, 32), (0, 64), (0, 100), (64, 128)])
@pytest.mark.parametrize("sm_scale", [0.0, 1.0])
def test_pipelined_attention_over_keys_of_weight_zero(d, n_q, lo, hi, sm_scale):
    S, H, cached, dtype = 4, 75, 110, torch.bfloat16
    kv = cached + n_q
    print(f"weight zero, pipelined d={d} n_q={n_q} keys {lo}..{hi} sm_scale={sm_scale}", flush=True)
    shape = skv.Shape(S, H, d, dtype, sm_scale)
    scale = sm_scale or d ** -0.5
    q, k, v = (_rand(94 + i, (S, H, n, d), dtype) for i, n in enumerate((n_q, kv, kv)))
    q = (q.float() / (scale * d ** 0.5)).to(dtype)
    q[..., 0] = 0.5
    keep = torch.ones(kv, dtype=torch.bool)
    keep[lo:hi] = False
    k[:, :, ~keep, 0] = float("-inf")
    pick = [0, S * H - 1]
    ref = oracle.attend(units(q)[pick], units(k)[pick][:, keep], units(v)[pick][:, keep], scale)
    dev = [t.contiguous().to(DEV) for t in (q, k, v, k[:, :, cached:], v[:, :, cached:], k[:, :, :cached], v[:, :, :cached])]
    out = torch.empty(S, H, n_q, d, dtype=dtype, device=DEV)
    skv.attend(shape, *dev[:3], kv, out)
    torch.cuda.synchronize()
    check_output(units(out)[pick], ref, dtype, "attend")
    kd, vd, out = torch.zeros_like(dev[1]), torch.zeros_like(dev[2]), torch.empty_like(out)
    skv.step(shape, dev[0], dev[3], dev[4], [0], dev[5], dev[6], cached, cached, kd, vd, out, None, None)
    torch.cuda.synchronize()
    check_output(units(out)[pick], ref, dtype, "step")
    assert torch.equal(kd, dev[1]) and torch.equal(vd, dev[2])


# a key of NaN makes the selectivity NaN, also where a lane holds no other key
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H", [(1, 2), (8, 16)])   # 128 units: the streamed route
def test_asi_of_a_key_of_nan(d, S, H):
    n_samp, hist, cur = 16, 512, 1
    print(f"asi of a key of NaN d={d} units={S * H}", flush=True)
    assert routes.asi_streams(torch.bfloat16, S * H, hist + cur, n_samp, 64) == (S * H == 128)
    shape = skv.Shape(S, H, d, torch.bfloat16)
    q, k = _rand(80, (S, H, n_samp, d), torch.bfloat16), _rand(81, (S, H, hist + cur, d), torch.bfloat16)
    k[:, :, -1] = float("nan")
    terms, mean = torch.zeros(S, H, n_samp, 2, device=DEV), torch.zeros(3, device=DEV)
    ws = torch.empty(skv.workspace_bytes(shape, hist + cur, n_samp), dtype=torch.uint8, device=DEV)
    skv.asi(shape, q.to(DEV), k.to(DEV), hist, cur, 64, terms, mean, ws)
    torch.cuda.synchronize()
    assert torch.isnan(terms).all() and torch.isnan(mean).all()


# arguments that the native marshalling leaves to the binding (a tensor subclass, NumPy integers in the Shape)
def test_prepared_steps_of_subclasses_and_numpy_integers():
    class Tagged(torch.Tensor):
        pass

    S, H, d, L, budget, n_cur, dtype = 1, 3, 64, 90, 20, 25, torch.bfloat16
    print("prepared calls with a tensor subclass", flush=True)
    q, kc, vc = (_rand(110 + i, (S, H, n_cur, d), dtype).to(DEV) for i in range(3))
    ks, vs = (_rand(113 + i, (S, H, L + n_cur, d), dtype).to(DEV) for i in range(2))
    win, win2 = list(range(n_cur - 16, n_cur)), [0, 7, 20]
    results = []
    for shape, cast in ((skv.Shape(S, H, d, dtype), lambda t: t),
                        (skv.Shape(np.int32(S), np.int64(H), np.int64(d), dtype), lambda t: t.as_subclass(Tagged))):
        ws = torch.empty(skv.workspace_bytes(shape, L + n_cur, n_cur), dtype=torch.uint8, device=DEV)
        kd, vd = (torch.zeros(S, H, budget + n_cur, d, dtype=dtype, device=DEV) for _ in range(2))
        kn, vn = (torch.zeros(S, H, budget + 3, d, dtype=dtype, device=DEV) for _ in range(2))
        cache = ks.clone(), vs.clone()
        out, out2 = torch.zeros_like(q), torch.zeros_like(q)
        step = skv.PreparedStep(shape, cast(q), kc, vc, win, cast(ks), vs, L, budget, cast(kd), vd, out, None, cast(ws))
        lit = skv.PreparedAppendFirst(shape, cast(q), kc, vc, win2, 3, cast(cache[0]), cache[1], L, budget, kn, cast(vn), out2,
                                      None, ws)
        assert step() == budget + n_cur and lit(torch.cuda.current_stream().cuda_stream) == budget + 3
        torch.cuda.synchronize()
        results.append((out, kd, vd, out2, kn, vn, *cache))
    assert float(results[0][0].abs().max()) > 0 and float(results[0][3].abs().max()) > 0
    for a, b in zip(*results):
        assert torch.equal(a, b)


# Kept rows are stored through the caches up to a size and past them beyond, by compact_kernel and by the ranking
# kernels: on either side of the limits, with a ragged end, every row of every unit.
@pytest.mark.parametrize("rows", [3051, 3053])
def test_large_compactions_on_both_sides_of_the_limit(rows):
    S, H, d, n_cur = 16, 16, 128, 7
    keep, L = rows - n_cur, rows + 200
    assert routes.rows_go_past_caches(False, S * H, rows, 2 * d) == (rows == 3053)
    print(f"compaction of {keep} + {n_cur} rows, {S * H} units", flush=True)
    shape = skv.Shape(S, H, d, torch.bfloat16)
    k, v = (torch.arange(S * H * L * d, device=DEV, dtype=torch.int32).mul_(m).to(torch.int16).view(torch.bfloat16).view(S, H, L, d)
            for m in (3, 5))
    kc, vc = (t[:, :, :n_cur].contiguous() for t in (v, k))
    idx = torch.randperm(L, generator=torch.Generator().manual_seed(rows))[:keep].sort().values.int().to(DEV)
    kd = torch.zeros(S, H, rows, d, dtype=torch.bfloat16, device=DEV)
    vd = torch.zeros_like(kd)
    skv.compact(shape, k, v, L, idx.expand(S, H, keep).contiguous(), keep, kc, vc, kd, vd)
    torch.cuda.synchronize()
    for got, cache, cur in ((kd, k, kc), (vd, v, vc)):   # (bits are compared: some are NaN)
        assert torch.equal(got[:, :, :keep].view(torch.int16), cache.view(torch.int16)[:, :, idx.long()])
        assert torch.equal(got[:, :, keep:].view(torch.int16), cur.view(torch.int16))


@pytest.mark.parametrize("keep", [1953, 1954])
def test_large_rankings_on_both_sides_of_the_limit(keep):
    S, H, d, L, n_cur = 16, 16, 128, 2100, 300
    assert routes.rows_go_past_caches(True, S * H, keep, 2 * d) == (keep == 1954)
    assert routes.step_kernel(torch.bfloat16, d, S * H, n_cur, L, keep) == "pipelined"
    print(f"ranking that keeps {keep} of {L} rows, {S * H} units", flush=True)
    shape = skv.Shape(S, H, d, torch.bfloat16)
    rand = lambda key, n: W.normal_tensor(W.stream_key(4321, key), (S, H, n, d), DEV).to(torch.bfloat16)
    q, kc, vc = (rand(60 + i, n_cur) for i in range(3))
    k, v = (rand(63 + i, L) for i in range(2))
    kd = torch.zeros(S, H, keep + n_cur, d, dtype=torch.bfloat16, device=DEV)
    vd, out = torch.zeros_like(kd), torch.empty_like(q)
    idx = torch.empty(S, H, keep, dtype=torch.int32, device=DEV)
    ws = torch.empty(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
    skv.step(shape, q, kc, vc, list(range(n_cur - 16, n_cur)), k, v, L, keep, kd, vd, out, idx, ws)
    torch.cuda.synchronize()
    assert bool((idx[..., 1:] > idx[..., :-1]).all()) and int(idx.min()) >= 0 and int(idx.max()) < L
    rows = idx.long()[..., None].expand(S, H, keep, d)
    for got, cache, cur in ((kd, k, kc), (vd, v, vc)):
        assert torch.equal(got[:, :, :keep], cache.gather(2, rows)) and torch.equal(got[:, :, keep:], cur)
