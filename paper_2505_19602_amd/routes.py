"""Which kernels a call takes, by its sizes: the dispatch rules of csrc/common.h, csrc/asi.hip and
csrc/api.hip in Python, for reports (bench.py prices each kernel against its own work) and for tests
that are written for one kernel.  tests/test_dispatch_host.py compares them with the C++ rules.
Output tensors that overlap inputs take other routes and are not covered."""
from __future__ import annotations

import torch

COMPUTE_UNITS = 256
ATTEND, APPEND, KEEP_ALL, RANKED = range(4)   # enum class SmallWork


def small_tile_rows(dtype: torch.dtype, d: int, units: int, n_q: int, kv: int, work: int) -> int:
    """Query rows per workgroup of the kernel for small work, 0 where it is not taken."""
    if dtype != torch.bfloat16:
        return 0
    for rows in (16, 32, 64, 128):
        n_wg = units * -(-n_q // rows)
        if n_wg <= COMPUTE_UNITS:
            break
    else:
        return 16 if n_q <= 16 else 0
    if rows <= 32:
        return rows
    if rows == 128:
        return rows if work == RANKED and kv <= 320 else 0
    spare = n_wg <= COMPUTE_UNITS * 7 // 8
    pays = work == RANKED or (work == KEEP_ALL and (d == 64 or spare or n_q <= 64)) or \
        (work == APPEND and d == 64 and spare) or (work == ATTEND and d == 64 and kv >= 512)
    return rows if pays else 0


def attend_kernel(dtype: torch.dtype, d: int, units: int, n_q: int, kv: int, work: int = ATTEND) -> str:
    """"f32", "small" or "pipelined"; work: ATTEND for scalekv_attend, APPEND for scalekv_step_append_first."""
    if dtype == torch.float32:
        return "f32"
    return "small" if small_tile_rows(dtype, d, units, n_q, kv, work) else "pipelined"


def step_kernel(dtype: torch.dtype, d: int, units: int, n_cur: int, cache_len: int, budget: int) -> str:
    """The same for the attention of scalekv_step; "small" prunes and appends in the same launch."""
    keep = min(budget, cache_len)
    work = RANKED if 0 < keep < cache_len else KEEP_ALL if keep else APPEND
    return attend_kernel(dtype, d, units, n_cur, keep + n_cur, work)


def ranks_in_one_launch(dtype: torch.dtype, units: int, cache_len: int) -> bool:
    """Scores, selection and pruning of a unit by one workgroup (or inside the kernel for small work)."""
    return dtype == torch.bfloat16 and cache_len <= 12288 and (units >= 64 or cache_len <= 4096)


def asi_streams(dtype: torch.dtype, units: int, length: int, n_samp: int, top_k: int) -> bool:
    """Selectivity without a workspace of logits."""
    if dtype != torch.bfloat16 or top_k > 256:
        return False
    rows, keys = min(n_samp, 32), units * length
    if min(units, 256) * rows >= (1024 if units >= 128 else 2048):
        return True
    return keys >= 160000 if rows == 32 else keys >= 220000 if rows >= 8 else keys >= 800000 and length >= 3000
