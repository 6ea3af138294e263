"""scalekv_step_static (the entry point that allocates nothing) against scalekv_step: same
kernels, so every output must be bit-identical -- indices, compacted K/V, attention output --
on calls in a row that share the library's one scratch array, each on a smaller input than the last."""
import pytest
import torch

import paper_2505_19602_amd as skv
import workloads as W
from paper_2505_19602_amd import routes

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rand(key, shape, dtype):
    return W.normal_tensor(W.stream_key(777, key), shape, DEV).to(dtype)


def _both_ways(case, S, H, d, n_cur, L, budget, dtype, with_idx=True):
    shape = skv.Shape(S, H, d, dtype)
    q, kc, vc = (_rand(10 * case + i, (S, H, n_cur, d), dtype) for i in range(3))
    ks, vs = _rand(10 * case + 3, (S, H, L, d), dtype), _rand(10 * case + 4, (S, H, L, d), dtype)
    win = list(range(max(0, n_cur - 16), n_cur))
    keep = min(budget, L)
    ws = torch.zeros(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
    assert ws.numel() <= skv.STATIC_SCRATCH_BYTES
    res = []
    for static in (False, True):
        kd = torch.full((S, H, keep + n_cur + 3, d), 7.0, dtype=dtype, device=DEV); vd = torch.full_like(kd, 7.0)
        out = torch.full((S, H, n_cur, d), 7.0, dtype=dtype, device=DEV)
        idx = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV) if with_idx else None
        if static:
            before = torch.cuda.memory_allocated()
            new_len = skv.step_static(shape, q, kc, vc, win, ks, vs, L, budget, kd, vd, out, idx)
            assert torch.cuda.memory_allocated() == before        # torch's allocator was not asked for anything
        else:
            new_len = skv.step(shape, q, kc, vc, win, ks, vs, L, budget, kd, vd, out, idx, ws)
        torch.cuda.synchronize()
        assert new_len == keep + n_cur
        res.append((kd, vd, out, idx))
    for a, b, name in zip(res[0], res[1], ("k_dst", "v_dst", "out", "idx")):
        assert (a is None and b is None) or torch.equal(a, b), f"case {case}: {name} differs between scalekv_step and scalekv_step_static"
    kd, vd, out, idx = res[1]
    assert torch.all(kd[:, :, keep + n_cur:] == 7.0) and torch.all(vd[:, :, keep + n_cur:] == 7.0)
    assert torch.isfinite(out.float()).all()
    if with_idx:
        assert int(idx.min()) >= 0 and int(idx.max()) < L


def test_step_static_matches_step_on_two_calls_in_a_row():
    # whole steps in one launch, which leave the scratch alone; then fp32, small head: logits, statistics
    # and indices in the scratch
    print("step_static: 2x3 units, 300 queries, 700 cached rows, bf16", flush=True)
    _both_ways(1, 2, 3, 128, 300, 700, 250, torch.bfloat16)
    print("step_static: 1x2 units, 40 queries, 90 cached rows, bf16", flush=True)
    _both_ways(2, 1, 2, 128, 40, 90, 17, torch.bfloat16)
    print("step_static: 1x2 units, 33 queries, 150 cached rows, fp32 d64", flush=True)
    _both_ways(3, 1, 2, 64, 33, 150, 60, torch.float32)


@pytest.mark.parametrize("with_idx", [True, False])   # False: the index list is in the scratch as well
def test_step_static_finds_an_earlier_calls_scratch(with_idx):
    # every route that writes the scratch array, each call smaller than the one before: the ranking kernel with logits
    # beyond its registers, the ranking by several workgroups to a unit (statistics where the indices go later), logits,
    # statistics, scores and indices by launches of their own (few units, more than 4096 rows), the ranking kernel without
    # logits of its own (indices alone), and fp32
    for case, (S, H, d, n_cur, L, budget, dtype, ranking) in enumerate((
            (1, 130, 128, 300, 4400, 250, torch.bfloat16, "unit"), (1, 100, 64, 40, 4300, 17, torch.bfloat16, "unit"),
            (1, 64, 128, 300, 4400, 250, torch.bfloat16, "spread"), (1, 64, 64, 40, 4200, 17, torch.bfloat16, "spread"),
            (2, 3, 128, 300, 6100, 250, torch.bfloat16, "stages"), (1, 2, 64, 40, 4100, 17, torch.bfloat16, "stages"),
            (1, 5, 128, 40, 1700, 100, torch.bfloat16, "spread"), (1, 5, 128, 40, 900, 100, torch.bfloat16, "spread"),
            (5, 53, 128, 20, 90, 30, torch.bfloat16, "unit"),
            (1, 5, 64, 70, 2100, 400, torch.float32, "stages"), (1, 2, 128, 40, 200, 60, torch.float32, "stages"))):
        assert ranking == ("stages" if not routes.ranks_in_one_launch(dtype, S * H, L) else
                           "spread" if routes.step_spreads(dtype, d, S * H, n_cur, L, budget) else "unit")
        print(f"step_static: {S}x{H} units, {n_cur} queries, {L} cached rows, {dtype} d{d}", flush=True)
        _both_ways(10 + case, S, H, d, n_cur, L, budget, dtype, with_idx)


def test_step_static_refuses_shapes_beyond_its_scratch_and_needs_none_without_a_ranking():
    S, H, d, n_cur, dtype = 4, 8, 128, 16, torch.bfloat16
    shape = skv.Shape(S, H, d, dtype)
    L = 40000                                                     # 32 units x 40000 rows: ~92 MB of scratch
    assert skv.workspace_bytes(shape, L, n_cur) > skv.STATIC_SCRATCH_BYTES
    q, kc, vc = (_rand(90 + i, (S, H, n_cur, d), dtype) for i in range(3))
    ks = torch.zeros(S, H, L, d, dtype=dtype, device=DEV); vs = torch.zeros_like(ks)
    kd = torch.zeros(S, H, L + n_cur, d, dtype=dtype, device=DEV); vd = torch.zeros_like(kd)
    out = torch.zeros(S, H, n_cur, d, dtype=dtype, device=DEV)
    with pytest.raises(skv.ScaleKVError) as err:
        skv.step_static(shape, q, kc, vc, list(range(16)), ks, vs, L, 100, kd, vd, out, None)
    assert err.value.status == 3 and "static" in str(err.value)
    # keeping everything ranks nothing and uses no scratch: legal at any size
    assert skv.step_static(shape, q, kc, vc, [], ks, vs, L, L, kd, vd, out, None) == L + n_cur
    torch.cuda.synchronize()
    assert torch.equal(kd[:, :, L:], kc) and torch.equal(vd[:, :, L:], vc)
