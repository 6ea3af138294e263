"""Runs a fixed list of library calls on seeded inputs and returns (or saves) every output.

tests/test_gpu_wg_order.py runs it twice: in the test process with the library in the tree, and in
a child process whose SCALEKV_LIBRARY names the build that walks every grid backwards
(python -m paper_2505_19602_amd.build --variant reversed_order).  Not collected by pytest."""
import hashlib
import os
import sys

import numpy as np
import torch

DEV = "cuda"


def run_all():
    import paper_2505_19602_amd as skv
    import workloads as W
    from paper_2505_19602_amd import routes

    out = {"library": np.array(os.path.basename(skv.lib_path()))}

    def rand(key, shape, dtype):
        return W.normal_tensor(W.stream_key(4321, key), shape, DEV).to(dtype)

    def keep_np(name, t):
        t = t.detach().cpu()
        a = (t.view(torch.int16) if t.dtype == torch.bfloat16 else t).numpy().copy()
        out[name] = a if a.size < 1 << 23 else np.array(hashlib.sha256(a.tobytes()).hexdigest())

    # (tag, S, H, d, n_cur, cache_len, budget, dtype, attention kernel, how the cache is ranked: by a workgroup per
    # unit ("unit"; in front of the small kernel or, up to 1536 rows, inside it), by several ("spread"), in the launches
    # of the single stages ("stages") or not at all).  Whole steps in one launch (several workgroups to a unit), fp32,
    # rankings in front of the small kernel, after which it prunes or not; then the pipelined attention, which appends,
    # behind each form of the ranking kernel: in LDS, in registers, and with the rows beyond them in the workspace; its
    # three forms, both kinds of append in the plain and split ones, and copying a cache that is kept whole
    bf16, f32 = torch.bfloat16, torch.float32
    cases = [("one_launch", 3, 11, 128, 100, 900, 333, bf16, "small", "unit"),
             ("one_launch_ragged", 2, 20, 128, 150, 1500, 210, bf16, "small", "unit"),
             ("one_launch_d64", 2, 15, 64, 150, 1500, 210, bf16, "small", "unit"),
             ("small", 2, 3, 128, 36, 140, 50, bf16, "small", "unit"),
             ("d64", 2, 2, 64, 70, 260, 90, bf16, "small", "unit"),
             ("fp32", 1, 2, 64, 33, 150, 60, f32, "f32", "stages"),
             ("fp32_long", 2, 5, 64, 33, 2500, 300, f32, "f32", "stages"),
             ("long", 1, 2, 128, 130, 12600, 1000, bf16, "small", "stages"),
             ("registers_small", 2, 40, 128, 40, 1700, 300, bf16, "small", "unit"),
             ("spread_small", 3, 5, 128, 300, 900, 333, bf16, "small", "spread"),
             ("spread_small_ragged", 2, 4, 128, 400, 1500, 210, bf16, "small", "spread"),
             ("spread_small_long", 1, 6, 128, 40, 1700, 300, bf16, "small", "spread"),
             ("spread_small_d64", 2, 4, 64, 400, 1500, 210, bf16, "small", "spread"),
             ("spread_pipe", 1, 65, 128, 530, 1700, 300, bf16, "pipelined", "spread"),
             ("spread_pipe_far", 1, 65, 128, 530, 4300, 300, bf16, "pipelined", "spread"),
             ("spread_pipe_far_d64", 1, 65, 64, 530, 4300, 300, bf16, "pipelined", "spread"),
             ("pipe_short", 5, 52, 128, 150, 300, 77, bf16, "pipelined", "unit"),
             ("pipe_short_d64", 5, 52, 64, 40, 300, 77, bf16, "pipelined", "unit"),
             ("pipe_registers", 1, 130, 128, 300, 1700, 300, bf16, "pipelined", "unit"),
             ("pipe_registers_d64", 1, 65, 64, 530, 1700, 300, bf16, "pipelined", "unit"),
             ("pipe_far", 1, 130, 128, 300, 4300, 300, bf16, "pipelined", "unit"),
             ("pipe_far_d64", 1, 100, 64, 300, 4300, 300, bf16, "pipelined", "unit"),
             ("pipe_loop_d64", 5, 52, 64, 330, 300, 77, bf16, "pipelined", "unit"),
             ("pipe_split", 4, 10, 128, 430, 500, 120, bf16, "pipelined", "unit"),
             ("pipe_split_d64", 4, 10, 64, 430, 500, 120, bf16, "pipelined", "unit"),
             ("pipe_wide", 16, 16, 128, 200, 2100, 1860, bf16, "pipelined", "unit"),
             ("copy_loop", 5, 52, 128, 330, 300, 300, bf16, "pipelined", "none"),
             ("copy_split", 4, 10, 128, 430, 500, 500, bf16, "pipelined", "none"),
             ("copy_split_d64", 4, 10, 64, 430, 500, 500, bf16, "pipelined", "none"),
             ("copy_wide", 16, 16, 128, 200, 1860, 1860, bf16, "pipelined", "none")]
    forms = {"pipe_short": "plain", "pipe_loop_d64": "plain", "pipe_split": "split", "pipe_split_d64": "split", "pipe_wide": "wide",
             "copy_loop": "plain", "copy_split": "split", "copy_split_d64": "split", "copy_wide": "wide"}
    for c, (tag, S, H, d, n_cur, L, budget, dtype, kernel, ranking) in enumerate(cases):
        assert routes.step_kernel(dtype, d, S * H, n_cur, L, budget) == kernel, tag
        assert ranking == ("none" if budget >= L else "stages" if not routes.ranks_in_one_launch(dtype, S * H, L) else
                           "spread" if routes.step_spreads(dtype, d, S * H, n_cur, L, budget) else "unit"), tag
        assert tag not in forms or routes.pipe_form(d, S * H, n_cur, min(budget, L) + n_cur) == forms[tag], tag
        print(f"workgroup order: step {tag}: {S}x{H} units, {n_cur} queries, {L} cached rows", flush=True)
        shape = skv.Shape(S, H, d, dtype)
        q, kc, vc = (rand(10 * c + i, (S, H, n_cur, d), dtype) for i in range(3))
        ks, vs = rand(10 * c + 3, (S, H, L, d), dtype), rand(10 * c + 4, (S, H, L, d), dtype)
        win = list(range(max(0, n_cur - 16), n_cur))
        keep = min(budget, L)
        ws = torch.zeros(skv.workspace_bytes(shape, L, n_cur), dtype=torch.uint8, device=DEV)
        kd = torch.zeros((S, H, keep + n_cur, d), dtype=dtype, device=DEV); vd = torch.zeros_like(kd)
        o = torch.zeros((S, H, n_cur, d), dtype=dtype, device=DEV)
        idx = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV)
        skv.step(shape, q, kc, vc, win, ks, vs, L, budget, kd, vd, o, idx, ws)
        torch.cuda.synchronize()
        for name, t in (("k_dst", kd), ("v_dst", vd), ("out", o), ("idx", idx)):
            keep_np(f"step_{tag}_{name}", t)

        # the single stages on the same inputs
        scores = torch.zeros((S, H, L), dtype=torch.float32, device=DEV)
        skv.score(shape, q[:, :, -len(win):].contiguous(), ks, L, scores, ws)
        idx2 = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV)
        skv.select(shape, scores, L, budget, idx2)
        kd2 = torch.zeros((S, H, keep + n_cur, d), dtype=dtype, device=DEV); vd2 = torch.zeros_like(kd2)
        skv.compact(shape, ks, vs, L, idx2, keep, kc, vc, kd2, vd2)
        o2 = torch.zeros_like(o)
        skv.attend(shape, q, kd2, vd2, keep + n_cur, o2)
        torch.cuda.synchronize()
        for name, t in (("scores", scores), ("idx", idx2), ("k_dst", kd2), ("v_dst", vd2), ("out", o2)):
            keep_np(f"stages_{tag}_{name}", t)

    # the literal order of Sec. 3.3 (append, attend, rank with pooling and forced window rows), with both
    # attention kernels; 1700 rows: the ranking kernel that holds the logits in registers, and the ranking by several
    # workgroups to a unit
    for tag, H, L in (("", 3, 500), ("_pipe", 130, 200), ("_registers", 130, 1556), ("_spread", 6, 1556)):
        S, d, n_cur, budget, dtype = 2, 128, 144, 120, torch.bfloat16
        print(f"workgroup order: step_append_first {S}x{H} units, {L} cached rows", flush=True)
        assert routes.attend_kernel(dtype, d, S * H, n_cur, L + n_cur, routes.APPEND) == ("small" if H < 10 else "pipelined")
        assert routes.ranks_in_one_launch(dtype, S * H, L + n_cur)
        assert routes.rank_spreads(d, S * H, L + n_cur, False) == (tag == "_spread")
        shape = skv.Shape(S, H, d, dtype)
        q, kc, vc = (rand(900 + i, (S, H, n_cur, d), dtype) for i in range(3))
        cap = L + n_cur
        kcache, vcache = rand(903, (S, H, cap, d), dtype), rand(904, (S, H, cap, d), dtype)
        win = skv.window_centroids(12, 12)
        keep = len(win) + min(budget, L + n_cur - len(win))
        kn = torch.zeros((S, H, keep, d), dtype=dtype, device=DEV); vn = torch.zeros_like(kn)
        o = torch.zeros((S, H, n_cur, d), dtype=dtype, device=DEV)
        idx = torch.full((S, H, keep), -1, dtype=torch.int32, device=DEV)
        ws = torch.zeros(skv.workspace_bytes(shape, cap, n_cur), dtype=torch.uint8, device=DEV)
        skv.step_append_first(shape, q, kc, vc, win, 7, kcache, vcache, L, budget, kn, vn, o, idx, ws)
        torch.cuda.synchronize()
        for name, t in (("k_cache", kcache), ("k_next", kn), ("v_next", vn), ("out", o), ("idx", idx)):
            keep_np(f"literal{tag}_{name}", t)

    # Eq. 2 terms and position-only retention
    print("workgroup order: asi, select_positional", flush=True)
    hist, cur, d, dtype = 700, 256, 128, torch.bfloat16
    for tag, S, H in (("", 2, 2), ("_streamed", 8, 16)):
        assert routes.asi_streams(dtype, S * H, hist + cur, 16, 64) == bool(tag)
        shape = skv.Shape(S, H, d, dtype)
        k = rand(950, (S, H, hist + cur, d), dtype)
        qs = rand(951, (S, H, 16, d), dtype)
        ws = torch.zeros(skv.workspace_bytes(shape, hist + cur, 16), dtype=torch.uint8, device=DEV)
        terms = torch.zeros((S, H, 16, 2), dtype=torch.float32, device=DEV)
        asi_out = torch.zeros(3, dtype=torch.float32, device=DEV)
        skv.asi(shape, qs, k, hist, cur, 64, terms, asi_out, ws)
        torch.cuda.synchronize()
        keep_np(f"asi{tag}_terms", terms)
        keep_np(f"asi{tag}_out", asi_out)
    S, H = 2, 2
    shape = skv.Shape(S, H, d, dtype)
    idxp = torch.full((S, H, 80), -1, dtype=torch.int32, device=DEV)
    skv.select_positional(shape, 500, 16, 64, idxp)
    torch.cuda.synchronize()
    keep_np("positional_idx", idxp)
    return out


if __name__ == "__main__":
    np.savez(sys.argv[1], **run_all())
    print("workgroup order: worker done", flush=True)
