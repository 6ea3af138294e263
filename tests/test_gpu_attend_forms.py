"""The three forms of the pipelined bf16 attention kernel (four waves, eight waves on 256 rows, groups of waves that
split the keys) at the edges of their tiles, groups and stages, against the oracle; rows whose scores rise so far above
the first block's that the pass is repeated; the two-segment form with the append."""
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
    """One attention of S x H units; with `cached` as a step that keeps that many rows and appends the others."""
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
        rows = max(cached, 1)
        parts = [t.contiguous() for t in (k[:, :, cached:], v[:, :, cached:], k[:, :, :rows], v[:, :, :rows])]
        kd, vd = torch.zeros_like(k), torch.zeros_like(v)
        skv.step(shape, q, parts[0], parts[1], [0], parts[2], parts[3], cached, cached, kd, vd, out, None, None)
        assert torch.equal(kd, k) and torch.equal(vd, v)
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


# The first block's largest weight is 2^-60.  100 natural units above it, 144 binary ones, the pass stays as it is; at
# 126.5 weights are 2^122.5, above the checked 2^120; at 150 they are infinite.
@pytest.mark.parametrize("rise", [100.0, 126.5, 150.0])
@pytest.mark.parametrize("form,d,S,H,n_q,kv", [("split", 64, 4, 5, 430, 500), ("split", 128, 4, 5, 430, 500),
                                               ("wide", 128, 16, 16, 130, 2100), ("plain", 128, 15, 20, 40, 200)])
@pytest.mark.parametrize("last", [False, True])
def test_scores_far_above_the_first_block_in_each_form(form, d, S, H, n_q, kv, rise, last):
    _check(form, d, S, H, n_q, kv, 3, rise, kv - 1 if last else 100)


@pytest.mark.parametrize("form,d,S,H,n_q,cached", [("split", 64, 4, 10, 430, 101), ("split", 128, 4, 10, 430, 64),
                                                   ("split", 128, 4, 10, 430, 129), ("wide", 128, 16, 16, 200, 1999)])
def test_step_of_two_segments_in_each_form(form, d, S, H, n_q, cached):
    assert routes.step_kernel(BF16, d, S * H, n_q, cached, cached) == "pipelined"
    _check(form, d, S, H, n_q, cached + n_q, 4, cached=cached)


# more workgroups than the compute units hold at once, and the split form of head_dim 64: tiles are appended as they
# pass through the loop; one query tile and several, no kept rows, ragged tiles of both segments
@pytest.mark.parametrize("form,d,S,H,n_q,cached", [
    ("plain", 128, 20, 30, 96, 0), ("plain", 128, 20, 30, 97, 1), ("plain", 128, 20, 30, 128, 64),
    ("plain", 128, 20, 20, 190, 63), ("plain", 128, 20, 20, 193, 65), ("plain", 128, 15, 20, 385, 130),
    ("plain", 64, 20, 41, 65, 0), ("plain", 64, 20, 41, 127, 3), ("plain", 64, 20, 20, 191, 128),
    ("plain", 64, 20, 30, 258, 61),
    ("split", 64, 4, 10, 449, 0), ("split", 64, 4, 10, 385, 191), ("split", 64, 4, 10, 500, 1),
])
def test_append_of_passing_tiles(form, d, S, H, n_q, cached):
    assert routes.step_kernel(BF16, d, S * H, n_q, cached, cached) == "pipelined"
    _check(form, d, S, H, n_q, cached + n_q, 6, cached=cached)


# values whose products with weights around 2^-60 and below would be lost (2^-80, 2^-110), or nearly (2^-36); and none
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
