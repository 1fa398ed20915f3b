"""Timed cases of the library: what its users have it do, each through a
public entry point, from the smallest calls to the largest.

A case is a dict of plain values.  ``kind`` says which entry point it takes:

- ``solve``    ``fw_apsp`` / ``fw_apsp_i32``: distances in place;
- ``plan``     ``SolvePlan``: the same solve replayed as one captured graph;
- ``pred``     ``fw_apsp_pred``: distances and canonical last hops;
- ``widest``   ``fw_apsp_semiring``: widest paths (max-min);
- ``reach``    ``fw_transitive_closure_bits``: reachability on packed bits;
- ``batch``    ``BatchPlan``: many ragged graphs in one captured launch.

The solvers overwrite their matrix, so a program that keeps its graph copies
the weights into the matrix it solves in; a pass is that copy and the solve.
Graphs are the ones of the repository's benchmark and generators: Bernoulli
edges, integer weights (exact in every order of the sums), 0 on the diagonal.
"""
import math

import torch

from paper_1001_4108_amd import (I32_INF, BatchPlan, SolvePlan, fw_apsp, fw_apsp_i32,
                                 fw_apsp_pred, fw_apsp_semiring, fw_transitive_closure_bits)


def listed():
    return [
        # the smallest call: one graph that a single workgroup closes; latency
        {"name": "solve_f32_n48", "kind": "solve", "dtype": "f32", "n": 48},
        # the benchmark's small graph, solved again and again through a plan
        {"name": "plan_f32_n512", "kind": "plan", "dtype": "f32", "n": 512},
        # an ordinary graph whose size is no multiple of a tile
        {"name": "solve_f32_n1500", "kind": "solve", "dtype": "f32", "n": 1500},
        # the size of the ablation ladder and of most larger serving requests
        {"name": "solve_f32_n4096", "kind": "solve", "dtype": "f32", "n": 4096},
        # an odd size as a caller's own contiguous matrix has it: unaligned rows
        {"name": "solve_f32_n6001", "kind": "solve", "dtype": "f32", "n": 6001},
        # the headline workload
        {"name": "solve_f32_n16384", "kind": "solve", "dtype": "f32", "n": 16384},
        # integer distances with negative weights and no negative cycle
        {"name": "solve_i32_n8192", "kind": "solve", "dtype": "i32", "n": 8192},
        # the same graph when the paths themselves are wanted
        {"name": "pred_i32_n8192", "kind": "pred", "dtype": "i32", "n": 8192, "half": False},
        # paths over weights that are no integers
        {"name": "pred_f32_half_n3000", "kind": "pred", "dtype": "f32", "n": 3000, "half": True},
        # widest (bottleneck) paths
        {"name": "widest_f32_n8192", "kind": "widest", "dtype": "f32", "n": 8192},
        # reachability of a sparse digraph
        {"name": "reach_n16384", "kind": "reach", "dtype": "bits", "n": 16384},
        # the ragged batch: sizes log-uniform in [16, 512]
        {"name": "batch_f32_4096", "kind": "batch", "dtype": "f32", "count": 4096, "lo": 16,
         "hi": 512},
    ]


def _size(rng, lo, hi):
    n = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    # half of the sizes as multiples of 4 (16-byte rows), the rest as they fall
    return max(lo, n // 4 * 4) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "plan", "pred", "pred", "widest", "reach",
                       "batch"])
    if kind == "solve":
        dtype = rng.choice(["f32", "f32", "i32"])
        return {"kind": kind, "dtype": dtype,
                "n": _size(rng, 16, 14000 if dtype == "f32" else 10000)}
    if kind == "plan":
        return {"kind": kind, "dtype": rng.choice(["f32", "i32"]), "n": _size(rng, 64, 4096)}
    if kind == "pred":
        dtype = rng.choice(["f32", "i32"])
        half = dtype == "f32" and rng.random() < 0.5
        return {"kind": kind, "dtype": dtype, "n": _size(rng, 64, 6000 if half else 8192),
                "half": half}
    if kind == "widest":
        return {"kind": kind, "dtype": "f32", "n": _size(rng, 128, 10000)}
    if kind == "reach":
        return {"kind": kind, "dtype": "bits", "n": _size(rng, 256, 32768)}
    lo = rng.choice([16, 32, 64])
    return {"kind": kind, "dtype": rng.choice(["f32", "f32", "i32"]),
            "count": round(math.exp(rng.uniform(math.log(64), math.log(4096)))), "lo": lo,
            "hi": rng.randint(2 * lo, 512)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
ROWS = 2048  # rows drawn at a time


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _weights(case, seed):
    """The n x n weight matrix of a single-graph case."""
    n, kind, dtype = case["n"], case["kind"], case["dtype"]
    g = _generator(seed)
    f32 = dtype == "f32"
    absent = I32_INF if not f32 else -math.inf if kind == "widest" else math.inf
    out = torch.empty((n, n), dtype=torch.float32 if f32 else torch.int32, device="cuda")
    pot = None if f32 else torch.randint(-500, 501, (n,), generator=g, device="cuda",
                                         dtype=torch.int32)
    for r in range(0, n, ROWS):
        m = min(ROWS, n - r)
        edge = torch.rand((m, n), generator=g, device="cuda") < (0.3 if f32 else 0.2)
        w = torch.randint(1, 1001, (m, n), generator=g, device="cuda", dtype=torch.int32)
        if pot is not None:  # negative edges, every cycle's weight unchanged
            w += pot[r:r + m, None]
            w -= pot[None, :]
        w = w.to(out.dtype)
        if case.get("half"):
            w += 0.5
        out[r:r + m] = torch.where(edge, w, torch.full_like(w, absent))
    out.fill_diagonal_(0)
    return out


def _bit_words(case, seed):
    """Packed adjacency of a digraph with about 1.2 edges per vertex."""
    n = case["n"]
    words = (n + 31) // 32
    g = _generator(seed)
    m = int(1.2 * n)
    u = torch.randint(0, n, (m,), generator=g, device="cuda")
    v = torch.randint(0, n, (m,), generator=g, device="cuda")
    cell = torch.unique(u * n + v)  # each edge once, so its bit can be added
    u, v = cell // n, cell % n
    bits = torch.zeros(n * words, dtype=torch.int64, device="cuda")
    bits.index_add_(0, u * words + v // 32, torch.ones_like(v) << (v % 32))
    return torch.where(bits >= 1 << 31, bits - (1 << 32), bits).to(torch.int32).view(n, words)


def _batch_sizes(case):
    """The sizes of a ragged batch: log-uniform, in a fixed scattered order."""
    count, lo, hi = case["count"], case["lo"], case["hi"]
    step = math.log(hi / lo)
    return [min(hi, max(lo, round(lo * math.exp(step * ((g * 0.6180339887498949) % 1.0)))))
            for g in range(count)]


def _batch_weights(case, seed):
    """All graphs of a batch one behind the other, rows padded to 16 bytes:
    the flat weights and each graph's (offset, n, ld)."""
    sizes = _batch_sizes(case)
    place, total = [], 0
    for n in sizes:
        ld = (n + 3) // 4 * 4
        place.append((total, n, ld))
        total += (n * ld + 63) // 64 * 64
    g = _generator(seed)
    f32 = case["dtype"] == "f32"
    edge = torch.rand(total, generator=g, device="cuda") < 0.4
    w = torch.randint(1, 101, (total,), generator=g, device="cuda", dtype=torch.int32)
    w = w.to(torch.float32) if f32 else w
    w = torch.where(edge, w, torch.full_like(w, math.inf if f32 else I32_INF))
    for off, n, ld in place:
        w[off:off + n * ld:ld + 1] = 0
    return w, place


def _views(flat, place):
    return [flat.as_strided((n, n), (ld, 1), off) for off, n, ld in place]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        w, place = _batch_weights(case, seed)
        d = w.clone()
        return {"kind": kind, "w": w, "d": d, "plan": BatchPlan(_views(d, place))}
    w = _bit_words(case, seed) if kind == "reach" else _weights(case, seed)
    state = {"kind": kind, "n": case["n"], "w": w, "d": w.clone()}
    if kind == "plan":
        state["plan"] = SolvePlan(state["d"])
    if kind == "pred":
        state["p"] = torch.empty((case["n"], case["n"]), dtype=torch.int32, device="cuda")
    return state


def run(state):
    kind, d = state["kind"], state["d"]
    d.copy_(state["w"])
    if kind == "solve":
        return fw_apsp(d) if d.dtype == torch.float32 else fw_apsp_i32(d)
    if kind == "pred":
        return fw_apsp_pred(d, state["p"])
    if kind == "widest":
        return fw_apsp_semiring(d, "maxmin")
    if kind == "reach":
        return fw_transitive_closure_bits(d, state["n"])
    state["plan"].launch("graph")
    return d


def work(case):
    """One pass: the weights read and the result written once (twice where the
    last hops are written too); an add and a min, or an and and an or, per
    pair and vertex."""
    kind = case["kind"]
    if kind == "batch":
        sizes = _batch_sizes(case)
        return {"bytes": sum(8 * n * n for n in sizes), "flops": sum(2 * n ** 3 for n in sizes)}
    n = case["n"]
    if kind == "reach":
        return {"bytes": 8 * n * ((n + 31) // 32), "flops": 2 * n ** 3}
    return {"bytes": (12 if kind == "pred" else 8) * n * n, "flops": 2 * n ** 3}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by the plain triple loop
# ---------------------------------------------------------------------------
EXACT_MAX_N = 8192


def _triple_loop(d, join, keep):
    """d_ij <- keep(d_ij, join(d_ik, d_kj)) over k, on (..., n, n)."""
    n = d.shape[-1]
    tmp = torch.empty_like(d)
    for k in range(n):
        join(d[..., :, k:k + 1], d[..., k:k + 1, :], out=tmp)
        keep(d, tmp, out=d)
    return d


def exact(case, seed):
    kind = case["kind"]
    wide = torch.float64 if case["dtype"] == "f32" else torch.int64
    if kind == "reach" or case.get("n", 0) > EXACT_MAX_N:
        return None
    if kind == "batch":
        w, place = _batch_weights(case, seed)
        out = w.to(wide)
        absent = math.inf if wide == torch.float64 else I32_INF
        order = sorted(range(len(place)), key=lambda g: place[g][1])
        for s in range(0, len(order), 256):  # graphs of like size, padded together
            group = order[s:s + 256]
            m = max(place[g][1] for g in group)
            d = torch.full((len(group), m, m), absent, dtype=wide, device=w.device)
            d.diagonal(dim1=-2, dim2=-1).zero_()
            for x, g in enumerate(group):
                off, n, ld = place[g]
                d[x, :n, :n] = out.as_strided((n, n), (ld, 1), off)
            _triple_loop(d, torch.add, torch.minimum)
            for x, g in enumerate(group):
                off, n, ld = place[g]
                out.as_strided((n, n), (ld, 1), off).copy_(d[x, :n, :n])
        return out
    d = _weights(case, seed).to(wide)
    if kind == "widest":
        return _triple_loop(d, torch.minimum, torch.maximum)
    _triple_loop(d, torch.add, torch.minimum)
    return (d, None) if kind == "pred" else d
