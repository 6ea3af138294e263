"""The three forms of the pipelined bf16 attention kernel (four waves, eight waves on 256 rows, groups of waves that
split the keys) at the edges of their tiles, groups and stages, against the oracle; rows whose scores rise so far above
the first tile's that the pass is repeated; the two-segment form with the append."""
import os
import subprocess
import sys

import pytest
import torch

import oracle
import paper_2505_19602_amd as skv
import workloads as W
from paper_2505_19602_amd import routes
from parity_util import check_output, units

pytestmark = pytest.mark.gpu
DEV, BF16 = "cuda", torch.bfloat16


def _rand(key, shape):
    return W.normal_tensor(W.stream_key(777, key), shape, DEV).to(BF16)


def _check(form, d, S, H, n_q, kv, key, rise=0.0, rise_from=0, cached=None, value_scale=1.0):
    """One attention of S x H units; with `cached` as a step that keeps that many of one more cached rows (none of none) and
    appends the others."""
    assert routes.attend_kernel(BF16, d, S * H, n_q, kv) == "pipelined"
    assert routes.pipe_form(d, S * H, n_q, kv) == form
    print(f"{form} d={d} {S}x{H} units {n_q} queries {kv} keys rise={rise} from {rise_from} cached={cached}", flush=True)
    shape = skv.Shape(S, H, d, BF16)
    q, k, v = (_rand(10 * key + i, (S, H, n, d)) for i, n in enumerate((n_q, kv, kv)))
    v = v * value_scale
    if rise:
        q[..., 0] = 8.0
        k[..., 0] = 0.0
        k[:, :, rise_from:, 0] = rise * d ** 0.5 / 8.0
    out = torch.empty_like(q)
    if cached is None:
        skv.attend(shape, q, k, v, kv, out)
    else:
        # (a step that keeps every row would copy both segments: test_copy_of_passing_tiles)
        held = cached + 1 if cached else 0
        assert routes.step_kernel(BF16, d, S * H, n_q, held, cached) == "pipelined"
        kc, vc = k[:, :, cached:].contiguous(), v[:, :, cached:].contiguous()
        ks, vs = (_rand(10 * key + 5 + i, (S, H, cached + 1, d)) for i in range(2))
        if rise:
            ks[..., 0] = 0.0
        idx = torch.full((S, H, cached), -1, dtype=torch.int32, device=DEV)
        kd, vd = (torch.full((S, H, kv + 1, d), 7.0, dtype=BF16, device=DEV) for _ in range(2))
        ws = torch.empty(skv.workspace_bytes(shape, cached + 1, n_q), dtype=torch.uint8, device=DEV)
        skv.step(shape, q, kc, vc, [0, n_q - 1], ks, vs, held, cached, kd, vd, out, idx, ws)
        took = idx.long().unsqueeze(-1).expand(-1, -1, -1, d)
        k, v = (torch.cat([src.gather(2, took), cur], 2) for src, cur in ((ks, kc), (vs, vc)))
        if cached:
            assert idx.min() >= 0 and idx.max() <= cached and torch.all(idx.diff(dim=2) > 0)
        assert torch.equal(kd[:, :, :kv], k) and torch.equal(vd[:, :, :kv], v)
        assert torch.all(kd[:, :, kv:] == 7.0) and torch.all(vd[:, :, kv:] == 7.0)
    torch.cuda.synchronize()
    pick = sorted({0, S * H // 2, S * H - 1})
    rows = sorted({0, 31, 32, 127, 128, n_q // 2, n_q - 33, n_q - 1} & set(range(n_q)))
    take = lambda t: units(t.reshape(S * H, 1, *t.shape[2:])[pick])
    ref = oracle.attend(take(q)[:, rows], take(k), take(v), d ** -0.5)
    check_output(take(out)[:, rows].double() / value_scale, ref / value_scale, BF16, form)
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kv", [320, 321, 383, 384, 385, 449, 577, 640, 1023])
def test_split_form_at_tile_and_group_edges(d, kv):
    _check("split", d, 4, 5, 430, kv, kv)


@pytest.mark.parametrize("n_q,kv", [(129, 2048), (200, 2049), (256, 2111), (256, 2112), (161, 2177), (224, 2304)])
def test_wide_form_at_tile_and_stage_edges(n_q, kv):
    _check("wide", 128, 16, 16, n_q, kv, kv)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q,kv", [(20, 1), (129, 31), (100, 33), (128, 64), (33, 65), (200, 127), (129, 129), (64, 193)])
def test_plain_form_of_few_keys(d, n_q, kv):
    _check("plain", d, 15, 20, n_q, kv, kv)


# The first tile's largest weight is about 1 (2^4 at most, since the other channels differ).  60 natural units above it,
# 86.6 binary ones, the pass stays as it is; 78 are 112.5: above the split form's 2^100, below the 2^120 of the others;
# at 86, 124 binary units, those repeat too, and from 100 on, 144, weights are infinite.
@pytest.mark.parametrize("rise", [60.0, 78.0, 86.0, 100.0, 126.5, 150.0])
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100), ("plain", 128, 15, 20, 40, 200)])
@pytest.mark.parametrize("last", [False, True])
def test_scores_far_above_the_first_block_in_each_form(form, d, S, H, n_q, kv, rise, last):
    _check(form, d, S, H, n_q, kv, 3, rise, kv - 1 if last else 100)


@pytest.mark.parametrize("form,d,S,H,n_q,cached", [("split", 64, 4, 10, 430, 101), ("split", 128, 4, 10, 430, 64),
                                                   ("split", 128, 4, 10, 430, 129), ("wide", 128, 16, 16, 200, 1999),
                                                   ("split", 128, 4, 10, 430, 1), ("wide", 128, 16, 16, 129, 2048)])
@pytest.mark.parametrize("rise", [0.0, 150.0])   # 150: workgroups repeat their pass, and append as well
def test_step_of_two_segments_in_each_form(form, d, S, H, n_q, cached, rise):
    _check(form, d, S, H, n_q, cached + n_q, 4, rise, max(cached, 100), cached=cached)


# more workgroups than the compute units hold at once, and the split form of head_dim 64: tiles are appended as they
# pass through the loop; one query tile and several, no kept rows, ragged tiles of both segments, kept rows of fewer tiles
# than groups and of a number that the groups do not share evenly
@pytest.mark.parametrize("form,d,S,H,n_q,cached", [
    ("plain", 128, 20, 30, 96, 0), ("plain", 128, 20, 30, 97, 1), ("plain", 128, 20, 30, 128, 64),
    ("plain", 128, 20, 20, 190, 63), ("plain", 128, 20, 20, 193, 65), ("plain", 128, 15, 20, 385, 130),
    ("plain", 64, 20, 41, 65, 0), ("plain", 64, 20, 41, 127, 3), ("plain", 64, 20, 20, 191, 128),
    ("plain", 64, 20, 30, 258, 61),
    ("split", 64, 4, 10, 449, 0), ("split", 64, 4, 10, 385, 191), ("split", 64, 4, 10, 500, 1), ("split", 64, 4, 10, 385, 100),
    ("split", 64, 4, 10, 400, 257), ("split", 64, 4, 10, 430, 448),
])
@pytest.mark.parametrize("rise", [0.0, 150.0])
def test_append_of_passing_tiles(form, d, S, H, n_q, cached, rise):
    _check(form, d, S, H, n_q, cached + n_q, 6, rise, max(cached, 64), cached=cached)


# a step that keeps everything: the pipelined kernel reads the source cache and copies the tiles that pass into another
# one, with strides and rows of its own.  One query tile and several, more of them than tiles, ragged tiles of both
# segments, one tile in all, groups without a tile, rows that make workgroups repeat their pass
@pytest.mark.parametrize("form,d,S,H,n_q,cached", [
    ("plain", 128, 20, 30, 96, 1), ("plain", 128, 16, 16, 30, 260), ("plain", 128, 20, 20, 190, 63), ("plain", 128, 4, 65, 900, 65),
    ("plain", 64, 20, 41, 65, 130), ("plain", 64, 20, 20, 191, 127), ("plain", 64, 10, 20, 40, 200),
    ("wide", 128, 16, 16, 129, 1999), ("wide", 128, 16, 16, 200, 2048), ("wide", 128, 8, 16, 500, 1700), ("wide", 128, 8, 16, 2040, 1020), ("wide", 128, 8, 16, 2040, 1019),
    ("split", 128, 4, 32, 100, 700), ("split", 128, 4, 10, 600, 257), ("split", 64, 4, 50, 33, 1001), ("split", 64, 8, 16, 100, 320),
])
@pytest.mark.parametrize("rise", [0.0, 150.0])
def test_copy_of_passing_tiles(form, d, S, H, n_q, cached, rise):
    kv = cached + n_q
    assert routes.step_kernel(BF16, d, S * H, n_q, cached, cached) == "pipelined" and routes.pipe_form(d, S * H, n_q, kv) == form
    print(f"copies both: {form} d={d} {S}x{H} units {n_q} queries {cached} cached rise={rise}", flush=True)
    shape = skv.Shape(S, H, d, BF16)
    q, kc, vc, k1, v1 = (_rand(70 + i, (S, H, n, d)) for i, n in enumerate((n_q, n_q, n_q, cached + 1, cached + 5)))
    if rise:
        q[..., 0] = 8.0
        k1[..., 0] = 0.0
        kc[..., 0] = rise * d ** 0.5 / 8.0
    ks, vs = k1[:, :, :cached].clone(), v1[:, :, :cached].clone()
    k1[:, :, cached:], v1[:, :, cached:] = float("nan"), float("nan")
    kd = torch.full((S, H + 1, kv + 2, d), 7.0, dtype=BF16, device=DEV)[:, :H]
    vd = torch.full((S, H, kv + 7, d), 7.0, dtype=BF16, device=DEV)
    out, idx = torch.empty_like(q), torch.full((S, H, cached), -1, dtype=torch.int32, device=DEV)
    skv.step(shape, q, kc, vc, [0], k1, v1, cached, cached, kd, vd, out, idx, None)
    torch.cuda.synchronize()
    k, v = torch.cat([ks, kc], 2), torch.cat([vs, vc], 2)
    assert torch.equal(kd[:, :, :kv], k) and torch.equal(vd[:, :, :kv], v)
    assert torch.all(kd[:, :, kv:] == 7.0) and torch.all(vd[:, :, kv:] == 7.0)
    assert torch.equal(idx, torch.arange(cached, dtype=torch.int32, device=DEV).expand(S, H, cached))
    pick = sorted({0, S * H // 2, S * H - 1})
    rows = sorted({0, 31, 32, 127, 128, n_q // 2, n_q - 1} & set(range(n_q)))
    take = lambda t: units(t.reshape(S * H, 1, *t.shape[2:])[pick])
    check_output(take(out)[:, rows], oracle.attend(take(q)[:, rows], take(k), take(v), d ** -0.5), BF16, form)
    assert torch.isfinite(out).all()


# The same with out on top of the map's keys or values or of the source cache: the kernel must not read (and copy) what
# other workgroups store their results over, so that the cache is written before.
@pytest.mark.parametrize("over", ["k_cur", "v_cur", "k_src", "v_src"])
@pytest.mark.parametrize("form,d,S,H,n_q,cached", [
    ("plain", 128, 10, 13, 300, 40), ("plain", 64, 20, 20, 191, 200), ("split", 128, 4, 10, 600, 257), ("split", 64, 8, 16, 100, 320),
    ("wide", 128, 8, 16, 500, 1700),
])
def test_copy_of_passing_tiles_under_the_output(form, d, S, H, n_q, cached, over):
    kv = cached + n_q
    assert routes.step_kernel(BF16, d, S * H, n_q, cached, cached) == "pipelined" and routes.pipe_form(d, S * H, n_q, kv) == form
    assert form != "wide" or 2 * cached >= n_q   # the sizes at which that form copies both segments
    print(f"copies both under out over {over}: {form} d={d} {S}x{H} units {n_q} queries {cached} cached", flush=True)
    shape = skv.Shape(S, H, d, BF16)
    q, kc, vc = (_rand(130 + i, (S, H, n_q, d)) for i in range(3))
    ks, vs = (_rand(133 + i, (S, H, max(cached, n_q), d)) for i in range(2))
    k, v = torch.cat([ks[:, :, :cached], kc], 2), torch.cat([vs[:, :, :cached], vc], 2)
    out = {"k_cur": kc, "v_cur": vc, "k_src": ks, "v_src": vs}[over].view(-1)[:q.numel()].view_as(q)
    kd, vd = (torch.full((S, H, kv + 1, d), 7.0, dtype=BF16, device=DEV) for _ in range(2))
    skv.step(shape, q, kc, vc, [0], ks, vs, cached, cached, kd, vd, out, None, None)
    torch.cuda.synchronize()
    assert torch.equal(kd[:, :, :kv], k) and torch.equal(vd[:, :, :kv], v)
    assert torch.all(kd[:, :, kv:] == 7.0) and torch.all(vd[:, :, kv:] == 7.0)
    pick = sorted({0, S * H // 2, S * H - 1})
    take = lambda t: units(t.reshape(S * H, 1, *t.shape[2:])[pick])
    rows = sorted({0, 31, n_q // 2, n_q - 1})
    check_output(take(out)[:, rows], oracle.attend(take(q)[:, rows], take(k), take(v), d ** -0.5), BF16, form)


# values whose products with weights far below 1 would be lost; and none
@pytest.mark.parametrize("value_scale", [2.0 ** -36, 2.0 ** -80, 2.0 ** -110])
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100), ("plain", 128, 15, 20, 40, 200)])
def test_small_values_in_each_form(form, d, S, H, n_q, kv, value_scale):
    _check(form, d, S, H, n_q, kv, 5, value_scale=value_scale)


def test_values_of_zero():
    shape = skv.Shape(15, 20, 128, BF16)
    q, k = _rand(1, (15, 20, 40, 128)), _rand(2, (15, 20, 200, 128))
    v, out = torch.zeros_like(k), torch.ones_like(q)
    skv.attend(shape, q, k, v, 200, out)
    assert torch.equal(out, torch.zeros_like(out))


# A channel of tiny values beside ordinary ones, compared on its own scale.
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100), ("plain", 128, 15, 20, 40, 200)])
def test_channels_of_small_values_in_each_form(form, d, S, H, n_q, kv):
    assert routes.pipe_form(d, S * H, n_q, kv) == form
    print(f"{form} d={d} channels of small values", flush=True)
    shape = skv.Shape(S, H, d, BF16)
    q, k, v = (_rand(70 + i, (S, H, n, d)) for i, n in enumerate((n_q, kv, kv)))
    scale = torch.ones(d, device=DEV)
    scale[5::8] = 2.0 ** -100
    out = torch.empty_like(q)
    skv.attend(shape, q, k, v * scale.to(BF16), kv, out)
    torch.cuda.synchronize()
    ref = oracle.attend(units(q)[[0, S * H - 1]], units(k)[[0, S * H - 1]], units(v)[[0, S * H - 1]], d ** -0.5)
    got = units((out.double() / scale.double()).float())[[0, S * H - 1]]
    check_output(got, ref, BF16, form)


# Weighted values beyond fp32 although the weights, 2^49, are not: the accumulators' own check has to trigger.  And
# accumulators of 2^125 to 2^127, which the groups of the split form must not add up.
@pytest.mark.parametrize("rise,value_scale", [(34.0, 2.0 ** 100), (32.0, 2.0 ** 79)])
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100), ("plain", 128, 15, 20, 40, 200)])
@pytest.mark.parametrize("last", [False, True])
def test_large_values_in_each_form(form, d, S, H, n_q, kv, rise, value_scale, last):
    _check(form, d, S, H, n_q, kv, 8, rise, kv - 1 if last else 100, value_scale=value_scale)


# Split form: one group meets a score in its first tile (key 64) to which four keys of another group, far above that
# group's first tile, add 3 %.  Its factor in the join underflows if it is formed from the groups' offsets alone.
# The same with the four within the range of the pass: what the join drops is then less than 2^-24.
@pytest.mark.parametrize("d,unit,first,high,top", [(64, 1.0, 192, 124.5, 129.0), (128, 2.0 ** 0.5, 128, 88.0, 91.5),
                                                   (64, 1.0, 192, 66.0, 69.5), (128, 2.0 ** 0.5, 128, 47.0, 49.5)])
def test_join_of_groups_with_distant_offsets(d, unit, first, high, top):
    S, H, n_q, kv = 4, 5, 430, 500
    assert routes.pipe_form(d, S * H, n_q, kv) == "split"
    print(f"join d={d} {high * unit:.1f} below {top * unit:.1f}", flush=True)
    q, k, v = torch.zeros(S, H, n_q, d), torch.zeros(S, H, kv, d), _rand(90, (S, H, kv, d)).cpu().float()
    q[..., 0] = unit * d ** 0.5 if d == 64 else 16.0   # a score is unit times the key's first channel
    k[:, :, 64, 0] = top
    high_rows = [first, first + 8, first + 16, first + 24]
    k[:, :, high_rows, 0] = high
    v[:, :, 64], v[:, :, high_rows] = -2.0, 2.0
    q, k, v = (t.to(BF16).to(DEV) for t in (q, k, v))
    out = torch.empty_like(q)
    skv.attend(skv.Shape(S, H, d, BF16), q, k, v, kv, out)
    torch.cuda.synchronize()
    ref = oracle.attend(units(q)[[0]], units(k)[[0]], units(v)[[0]], d ** -0.5)
    assert (ref[0, 0] + 2.0).max() > 0.04   # what the four keys add is seen
    check_output(units(out)[[0]], ref, BF16, "join")


# A score of the first tile, 64 keys, that lies far above the others is the exponent offset: its weight is 1 without
# rounding.  Keys a and b, both in its second half, outweigh all others by 2^45 and more, b with 0.7503 of a's weight, which bf16 rounds to
# 0.75: with values 0.75 and -1 they cancel exactly.  With any other offset, such as the maximum over the first block,
# both weights are rounded, and 1e-4 to 1e-3 is left in most rows.
@pytest.mark.parametrize("form,d,S,H,n_q,kv,a,b", [
    ("split", 64, 4, 5, 430, 500, 40, 63), ("split", 128, 4, 5, 430, 500, 32, 41), ("wide", 128, 16, 16, 130, 2100, 63, 47),
    ("plain", 128, 15, 20, 40, 200, 33, 60), ("plain", 64, 15, 20, 40, 64, 50, 34), ("plain", 128, 15, 20, 40, 37, 36, 35)])
def test_largest_weight_of_the_first_tile_is_one(form, d, S, H, n_q, kv, a, b):
    assert routes.pipe_form(d, S * H, n_q, kv) == form
    print(f"{form} d={d} {kv} keys, largest weights at {a} and {b}", flush=True)
    q, k, v = torch.zeros(S, H, n_q, d), torch.zeros(S, H, kv, d), torch.zeros(S, H, kv, d)
    q[..., 0], q[..., 1] = 44.0 + 0.25 * (torch.arange(n_q) % 32), 1.0
    k[:, :, [a, b], 0] = 8.0
    k[:, :, b, 1] = -2.296875 if d == 64 else -3.25   # ln 0.7503 = -0.2873
    v[:, :, a], v[:, :, b] = 0.75, -1.0
    q, k, v = (t.to(BF16).to(DEV) for t in (q, k, v))
    out = torch.empty_like(q)
    skv.attend(skv.Shape(S, H, d, BF16), q, k, v, kv, out)
    torch.cuda.synchronize()
    ref = oracle.attend(units(q)[[0]], units(k)[[0]], units(v)[[0]], d ** -0.5)
    check_output(units(out)[[0]], ref, BF16, form)
    assert out.abs().max() < 1e-6


# Keys whose logits are all -inf have weight zero: a first block, a first tile, tiles further on, and every tile of one
# group (split form: tiles 1, 3, 5, 7, head_dim 64: 1, 4, 7), which then has nothing to join.
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100)])
@pytest.mark.parametrize("where", ["first_block", "first_tile", "two_tiles", "group", "rest"])
def test_keys_of_weight_zero_in_each_form(form, d, S, H, n_q, kv, where):
    assert routes.pipe_form(d, S * H, n_q, kv) == form
    print(f"weight zero, {form} d={d} {where}", flush=True)
    tile, groups = torch.arange(kv) // 64, 3 if d == 64 else 2
    gone = {"first_block": torch.arange(kv) < 32, "first_tile": tile == 0, "two_tiles": (tile == 1) | (tile == 2),
            "group": tile % groups == 1, "rest": tile > 0}[where]
    q, k, v = (_rand(120 + i, (S, H, n, d)) for i, n in enumerate((n_q, kv, kv)))
    q[..., 0] = 0.5
    k[:, :, gone.to(DEV), 0] = float("-inf")
    out = torch.empty_like(q)
    skv.attend(skv.Shape(S, H, d, BF16), q, k, v, kv, out)
    torch.cuda.synchronize()
    pick = [0, S * H - 1]
    ref = oracle.attend(units(q)[pick], units(k)[pick][:, ~gone], units(v)[pick][:, ~gone], d ** -0.5)
    check_output(units(out)[pick], ref, BF16, form)
    assert torch.isfinite(out).all()


# The measurement-only build without tile transfers fetches the tiles that fill its stages once: with no more keys than
# that it computes what the library does.
NO_TRANSFER = os.path.join(os.path.dirname(skv.__file__), "libscalekv_no_transfer.so")
NO_TRANSFER_CHILD = """
import sys, torch
import paper_2505_19602_amd as skv
q, k, v = torch.load(sys.argv[1], weights_only=True)
q, k, v = q.cuda(), k.cuda(), v.cuda()
out = torch.empty_like(q)
skv.attend(skv.Shape(15, 20, q.shape[3], torch.bfloat16), q, k, v, k.shape[2], out)
torch.save(out.cpu(), sys.argv[2])
"""


@pytest.mark.skipif(not os.path.exists(NO_TRANSFER),
                    reason="build it with: python -m paper_2505_19602_amd.build --variant no_transfer")
@pytest.mark.parametrize("d", [64, 128])
def test_build_without_transfers_fills_its_stages(d, tmp_path):
    assert routes.pipe_form(d, 300, 40, 128) == "plain"
    print(f"no_transfer build d={d}", flush=True)
    q, k, v = (_rand(80 + i, (15, 20, n, d)) for i, n in enumerate((40, 128, 128)))
    out = torch.empty_like(q)
    skv.attend(skv.Shape(15, 20, d, BF16), q, k, v, 128, out)
    torch.save([t.cpu() for t in (q, k, v)], tmp_path / "in.pt")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, SCALEKV_LIBRARY=NO_TRANSFER, PYTHONPATH=root + os.pathsep + os.environ.get("PYTHONPATH", ""))
    res = subprocess.run([sys.executable, "-c", NO_TRANSFER_CHILD, str(tmp_path / "in.pt"), str(tmp_path / "out.pt")], env=env,
                         capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-2000:]
    assert torch.equal(out.cpu(), torch.load(tmp_path / "out.pt", weights_only=True))
