"""What a program built on this library has it do, as cases that can be timed.

A case is one pass through the public entry points on device-resident tensors: one ScaleKV step
(`step`), the prepared steps of one layer through every scale of an image (`layer`), one step in
the literal order of the paper's selection (`literal`), one step of a position-only policy
(`positional`), or the attention selectivity of one layer at one scale (`asi`).  Sizes come from
the workload table of this repository (batch 1 at 512^2, batch 8 with guidance rows at 1024^2, the
wider 40-layer shape) and from ragged maps in between.
"""
from __future__ import annotations

import math

import torch

import paper_2505_19602_amd as skv

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
SIDES = (1, 2, 4, 6, 8, 12, 16, 20, 24, 32, 40, 48, 64)  # side lengths of an image's token maps
WINDOW = 16
MAX_FLOPS = 5.7e12  # the work of the largest listed case


def _step(name, seqs, heads, dim, dtype, cache, budget, rows, cols, values):
    return {"name": name, "kind": "step", "seqs": seqs, "heads": heads, "dim": dim, "dtype": dtype,
            "cache": cache, "budget": budget, "rows": rows, "cols": cols, "values": values}


def listed():
    return [
        # the third map of one 512^2 image: a few rows, the call itself is the cost
        _step("first_maps_batch1", 1, 16, 128, "bf16", 69, 14, 4, 4, "lowrank"),
        # a layer of one 512^2 image through its ten maps, budget 20 %: interactive generation
        {"name": "layer_512_batch1", "kind": "layer", "seqs": 1, "heads": 16, "dim": 128, "dtype": "bf16",
         "prefix": 64, "maps": 10, "percent": 20, "values": "lowrank"},
        # a refiner layer of eight 1024^2 images with guidance rows through its thirteen maps
        {"name": "layer_1024_batch16", "kind": "layer", "seqs": 16, "heads": 16, "dim": 128, "dtype": "bf16",
         "prefix": 64, "maps": 13, "percent": 5, "values": "lowrank"},
        # a map in the middle of that image (24 x 24), drafter budget
        _step("middle_map_batch16", 16, 16, 128, "bf16", 546, 246, 24, 24, "lowrank"),
        # its last map, drafter budget: where most of the time goes
        _step("last_map_drafter", 16, 16, 128, "bf16", 3350, 1622, 64, 64, "lowrank"),
        # the last map of the wider model, refiner budget, heavy-tailed keys
        _step("last_map_wide_refiner", 16, 32, 128, "bf16", 2516, 328, 64, 64, "heavy"),
        # the last map with nothing evicted: the uncompressed attention that users compare against
        _step("last_map_uncompressed", 16, 16, 128, "bf16", 6489, 6489, 64, 64, "lowrank"),
        # a map that is not square, an odd number of cached rows, narrow heads
        _step("ragged_map_narrow_heads", 3, 20, 64, "bf16", 1733, 433, 27, 45, "lowrank"),
        # full precision, as when results are checked against the bf16 run
        _step("map_f32", 2, 16, 128, "f32", 585, 117, 20, 20, "lowrank"),
        # the literal order with patch-centroid window and pooled scores
        {"name": "literal_map_48", "kind": "literal", "seqs": 16, "heads": 16, "dim": 128, "dtype": "bf16",
         "cache": 1809, "budget": 1046, "rows": 48, "cols": 48, "pool": 7, "values": "lowrank"},
        # sinks and most recent rows instead of scores, batch 2 with guidance rows
        {"name": "sinks_and_recent_map_32", "kind": "positional", "seqs": 4, "heads": 16, "dim": 128,
         "dtype": "bf16", "cache": 765, "sinks": 16, "recent": 140, "rows": 32, "cols": 32, "values": "lowrank"},
        # calibration: attention selectivity of one layer at the last map against the full history
        {"name": "asi_last_map", "kind": "asi", "seqs": 16, "heads": 16, "dim": 128, "dtype": "bf16",
         "cache": 6489, "rows": 64, "cols": 64, "samples": 16, "top": 64, "values": "lowrank"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        kind = rng.choice(("step", "step", "step", "step", "step", "step", "layer", "layer", "literal", "positional",
                           "asi", "f32"))
        case = {"kind": "step" if kind == "f32" else kind, "seqs": _log_int(rng, 1, 16),
                "heads": rng.choice((8, 12, 16, 20, 24, 32)), "dim": rng.choice((128, 128, 128, 64)),
                "dtype": "f32" if kind == "f32" else "bf16", "values": rng.choice(("lowrank", "lowrank", "heavy"))}
        if kind == "layer":
            case.update(prefix=_log_int(rng, 16, 128), maps=rng.randint(4, 13), percent=rng.randint(4, 25))
        else:
            area = _log_int(rng, 1, 700 if kind == "f32" else 4096)
            rows = max(1, int(round(math.sqrt(area) * rng.uniform(0.7, 1.0))))
            cols = max(1, min(area // rows, 4096 // rows))
            cache = _log_int(rng, 16, 1200 if kind == "f32" else 6489)
            case.update(rows=rows, cols=cols, cache=cache)
            if kind == "positional":
                sinks = rng.choice((0, 4, 16))
                case.update(sinks=sinks, recent=max(1, int(cache * rng.uniform(0.04, 0.25)) - sinks))
            elif kind == "asi":
                case.update(samples=min(rows * cols, rng.choice((8, 16, 32, 64))), top=rng.choice((16, 64, 128)))
            else:
                part = rng.choice((rng.uniform(0.04, 0.5), rng.uniform(0.04, 0.5), rng.uniform(0.04, 0.5), 1.0))
                case.update(budget=max(1, int(cache * part)))
                if kind == "literal":
                    case.update(pool=rng.choice((1, 3, 7)))
        most = MAX_FLOPS / 100 if kind == "f32" else MAX_FLOPS
        if work(case)["flops"] <= most:
            return case


# ---- the cases' own arithmetic: how many rows a layer's calls see

def _maps(case):
    """(map rows, cached rows, budget) of each call of a layer: everything is kept at the first two maps."""
    calls, cached, full = [], case["prefix"], case["prefix"]
    for k, side in enumerate(SIDES[: case["maps"]]):
        budget = full if k < 2 else max(1, int(full * case["percent"] / 100 + 0.5))
        calls.append((side * side, cached, budget))
        cached = min(budget, cached) + side * side
        full += side * side
    return calls


def _step_work(case, n, cached, budget):
    units, d, e = case["seqs"] * case["heads"], case["dim"], 4 if case["dtype"] == "f32" else 2
    keep = min(budget, cached)
    ranks = 0 < keep < cached
    reads = 3 * n + (cached if ranks else keep) + keep      # q, k, v of the map; keys and kept values of the cache
    writes = n + 2 * (keep + n)                             # output, new cache
    flops = 4 * n * (keep + n) * d + (2 * min(WINDOW, n) * cached * d if ranks else 0)
    return units * (reads + writes) * d * e, units * flops


def work(case):
    units, d, e = case["seqs"] * case["heads"], case["dim"], 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "layer":
        each = [_step_work(case, *call) for call in _maps(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    n, cached = case["rows"] * case["cols"], case["cache"]
    if case["kind"] == "step":
        moved, flops = _step_work(case, n, cached, case["budget"])
    elif case["kind"] == "literal":
        win = min(4, case["rows"]) * min(4, case["cols"])
        total = cached + n
        keep = win + min(case["budget"], total - win)
        kept = 2 * keep if keep < total else 0
        moved = units * (2 * cached + 3 * n + 3 * n + kept) * d * e + units * keep * 4
        flops = units * (4 * n * total * d + (2 * win * total * d if kept else 0))
    elif case["kind"] == "positional":
        sinks = min(case["sinks"], cached)
        keep = sinks + min(case["recent"], cached - sinks)
        moved = units * (2 * keep + 3 * n + n + 2 * (keep + n)) * d * e + units * keep * 4
        flops = units * 4 * n * (keep + n) * d
    else:
        moved = units * (cached + n + case["samples"]) * d * e + units * case["samples"] * 8
        flops = units * 2 * case["samples"] * (cached + n) * d
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    if case["kind"] == "asi":
        return {"rel": 2e-5}  # fp32 sums of exponentials over fp32 logits
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2, "max": 0.1}  # bf16 outputs, probabilities rounded to bf16; cache rows are copies


# ---- inputs

def _normal(gen, *size):
    return torch.randn(*size, device="cuda", dtype=torch.float32, generator=gen)


class _Values:
    """Queries, keys and values of one layer: `lowrank` shares a rank-8 subspace per head between
    queries and keys (peaked attention), `heavy` has Student-t keys."""

    def __init__(self, case, seed):
        self.case, self.dtype = case, DTYPES[case["dtype"]]
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.w = _normal(self.gen, case["heads"], 8, case["dim"]) / math.sqrt(8.0)
        self.wv = _normal(self.gen, case["heads"], 8, case["dim"]) / math.sqrt(8.0)

    def _size(self, n):
        return self.case["seqs"], self.case["heads"], n, self.case["dim"]

    def _mixed(self, n, w):
        x = _normal(self.gen, *self._size(n))
        if self.case["values"] == "lowrank":
            x += torch.matmul(_normal(self.gen, self.case["seqs"], self.case["heads"], n, 8), w)
        return x.to(self.dtype)

    def q(self, n):
        return self._mixed(n, self.w)

    def k(self, n):
        if self.case["values"] == "lowrank":
            return self._mixed(n, self.w)
        x = _normal(self.gen, *self._size(n))
        chi = sum(_normal(self.gen, *self._size(n)).square_() for _ in range(3))
        return (x / torch.sqrt(chi)).to(self.dtype)

    def v(self, n):
        return self._mixed(n, self.wv)

    def empty(self, n):
        return torch.empty(self._size(n), device="cuda", dtype=self.dtype)


def _workspace(shape, cached, n):
    return torch.empty(skv.workspace_bytes(shape, cached, n), dtype=torch.uint8, device="cuda")


def _last(n):
    return list(range(max(0, n - WINDOW), n))


def prepare(case, seed):
    values = _Values(case, seed)
    shape = skv.Shape(case["seqs"], case["heads"], case["dim"], values.dtype)
    state = {"kind": case["kind"], "shape": shape}
    if case["kind"] == "layer":
        calls = _maps(case)
        room = max(min(budget, cached) + n for n, cached, budget in calls)
        prefix = values.k(case["prefix"]), values.v(case["prefix"])
        pair = [(values.empty(room), values.empty(room)) for _ in range(2)]
        ws = _workspace(shape, max(cached for _, cached, _ in calls), max(n for n, _, _ in calls))
        src, state["calls"], state["out"] = prefix, [], []
        for i, (n, cached, budget) in enumerate(calls):
            q, k, v, out = values.q(n), values.k(n), values.v(n), values.empty(n)
            state["calls"].append(skv.PreparedStep(shape, q, k, v, _last(n), src[0], src[1], cached, budget,
                                                   pair[i % 2][0], pair[i % 2][1], out, None, ws))
            state["out"].append(out)
            src = pair[i % 2]
        length = min(calls[-1][2], calls[-1][1]) + calls[-1][0]
        state["k"], state["v"] = src[0][:, :, :length], src[1][:, :, :length]
        return state
    n, cached = case["rows"] * case["cols"], case["cache"]
    if case["kind"] == "asi":
        state.update(q=values.q(case["samples"]), k=values.k(cached + n), hist=cached, cur=n, top=case["top"],
                     terms=torch.empty(case["seqs"], case["heads"], case["samples"], 2, device="cuda"),
                     asi=torch.empty(3, device="cuda"), ws=_workspace(shape, cached + n, case["samples"]))
        return state
    state.update(q=values.q(n), k_cur=values.k(n), v_cur=values.v(n), out=values.empty(n), cached=cached)
    if case["kind"] == "literal":
        window = skv.window_centroids(case["rows"], case["cols"])
        total = cached + n
        keep = len(window) + min(case["budget"], total - len(window))
        state.update(k_src=values.k(total), v_src=values.v(total), k=values.empty(keep), v=values.empty(keep),
                     window=window, pool=case["pool"], budget=case["budget"], ws=_workspace(shape, total, n),
                     idx=torch.empty(case["seqs"], case["heads"], keep, dtype=torch.int32, device="cuda"))
        if keep == total:  # everything is kept: the cache stays where it is
            state.update(k=None, v=None)
        return state
    state.update(k_src=values.k(cached), v_src=values.v(cached))
    if case["kind"] == "positional":
        sinks = min(case["sinks"], cached)
        keep = sinks + min(case["recent"], cached - sinks)
        state.update(k=values.empty(keep + n), v=values.empty(keep + n), sinks=case["sinks"], recent=case["recent"],
                     idx=torch.empty(case["seqs"], case["heads"], keep, dtype=torch.int32, device="cuda"))
        return state
    keep = min(case["budget"], cached)
    state.update(k=values.empty(keep + n), v=values.empty(keep + n), window=_last(n), budget=case["budget"],
                 ws=_workspace(shape, cached, n))
    return state


def run(state):
    s = state
    if s["kind"] == "layer":
        for call in s["calls"]:
            call()
        return {"out": s["out"], "k": s["k"], "v": s["v"]}
    if s["kind"] == "step":
        skv.step(s["shape"], s["q"], s["k_cur"], s["v_cur"], s["window"], s["k_src"], s["v_src"], s["cached"],
                 s["budget"], s["k"], s["v"], s["out"], None, s["ws"])
        return {"out": s["out"], "k": s["k"], "v": s["v"]}
    if s["kind"] == "literal":
        skv.step_append_first(s["shape"], s["q"], s["k_cur"], s["v_cur"], s["window"], s["pool"], s["k_src"],
                              s["v_src"], s["cached"], s["budget"], s["k"], s["v"], s["out"], s["idx"], s["ws"])
        return {"out": s["out"], "k": s["k"], "v": s["v"], "idx": s["idx"], "k_cache": s["k_src"],
                "v_cache": s["v_src"]}
    if s["kind"] == "positional":
        keep = skv.select_positional(s["shape"], s["cached"], s["sinks"], s["recent"], s["idx"])
        length = skv.compact(s["shape"], s["k_src"], s["v_src"], s["cached"], s["idx"], keep, s["k_cur"], s["v_cur"],
                             s["k"], s["v"])
        skv.attend(s["shape"], s["q"], s["k"], s["v"], length, s["out"])
        return {"out": s["out"], "k": s["k"], "v": s["v"], "idx": s["idx"]}
    skv.asi(s["shape"], s["q"], s["k"], s["hist"], s["cur"], s["top"], s["terms"], s["asi"], s["ws"])
    return {"terms": s["terms"], "asi": s["asi"]}
