"""Sizes at which a kernel or a rule of its dispatch can go wrong: edges of tiles, remainders, the
smallest and largest of a range.  Everything is compared with the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_19602_amd as skv
import workloads as W
from parity_util import check_output, units

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rand(key, shape, dtype, scale=1.0):
    return (W.normal_tensor(W.stream_key(4321, key), shape) * scale).to(dtype)


# 16 and 32 query rows per wave (many units), 1, 2 and 4 waves sharing the keys, a wave without keys,
# ragged blocks of 16 keys and of query rows
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("S,H,n_q,kv_len", [
    (1, 2, 1, 1), (1, 2, 16, 15), (1, 3, 17, 16), (2, 2, 15, 17), (1, 2, 33, 48), (1, 2, 40, 63), (1, 2, 5, 65),
    (1, 1, 31, 129), (4, 48, 64, 33), (4, 48, 50, 80), (1, 100, 120, 20),
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
