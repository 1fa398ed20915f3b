"""The 128-wide diagonal launches of a batch: at most one tile per CU (256) and
more take closures of different geometries, with the same sums as a solve alone;
tiles of part of the matrix move in whole pieces.  Counts on both sides of the
line, the edges of pieces of two and four columns and of the 8-vertex sub-blocks,
the smallest matrices, rows of any alignment; and a launch with a CU per tile
takes no longer than one tile."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd import gen

pytestmark = pytest.mark.gpu


def _padded(w, pad, fill):
    n = w.shape[0]
    host = np.full((n, n + pad), fill, dtype=w.dtype)
    host[:, :n] = w
    t = torch.from_numpy(host).cuda()
    return t[:, :n], t


@pytest.mark.parametrize("count", [256, 257])
@pytest.mark.parametrize("n,pad", [(66, 0), (97, 1), (126, 2), (127, 0), (128, 3), (200, 0)])
def test_bits_of_a_solve_alone(n, pad, count):
    """Fractional fp32 weights, whose sums round."""
    rng = np.random.default_rng((n, count))
    w = gen.dense_graph(n, 0.4, 1, 50, seed=(n, pad)) + rng.random((n, n), dtype=np.float32)
    np.fill_diagonal(w, 0)
    alone = torch.from_numpy(w).cuda()
    batch = [_padded(w, pad, np.float32(7)) for _ in range(count)]
    try:
        fw.plan_set("f32", n, n, 128)
        fw.fw_apsp_plan(alone, 128)
        fw.fw_apsp_batched([v for v, _ in batch])
    finally:
        fw.plan_reset()
    for v, whole in batch:
        assert torch.equal(v.contiguous().view(torch.int32), alone.view(torch.int32))
        assert (whole[:, n:] == 7).all()


@pytest.mark.parametrize("dtype", [np.float32, np.int32])
@pytest.mark.parametrize("count", [300, 512, 513])
def test_sizes_that_differ(count, dtype):
    """Between a tile per CU and two, the sizes decide the form: here they differ
    (65 to 200), so 300 and 512 graphs' closures work ahead, in rounds, in both
    stages, and 513 graphs' do not."""
    sizes = [round(65 * (200 / 65) ** ((g * 0.6180339887498949) % 1)) for g in range(count)]
    code = "f32" if dtype == np.float32 else "i32"
    alone, batch = {}, []
    try:
        fw.plan_set(code, 65, 200, 128)
        for n in sorted(set(sizes)):
            w = gen.dense_graph(n, 0.3, 1, 50, seed=n, dtype=dtype)
            if dtype == np.float32:
                w += np.random.default_rng(n).random((n, n), dtype=np.float32)
                np.fill_diagonal(w, 0)
            src = torch.from_numpy(w).cuda()
            alone[n] = (src, fw.fw_apsp_plan(src.clone(), 128)[0])
        batch = [alone[n][0].clone() for n in sizes]
        fw.fw_apsp_batched(batch)
    finally:
        fw.plan_reset()
    for n, d in zip(sizes, batch):
        assert torch.equal(d.view(torch.int32), alone[n][1].view(torch.int32)), n


@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.int32])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 8, 9, 15, 23, 24, 25, 29, 30, 61, 63, 125, 126])
def test_part_of_a_tile(n, pad, dtype, tile):
    w = gen.dense_graph(n, 0.5, 1, 100, seed=(n, pad), dtype=dtype)
    v, whole = _padded(w, pad, dtype(7))
    fw.fw_apsp_plan(v, tile)
    assert np.array_equal(v.cpu().numpy(), oracle.fw(w))
    assert (whole[:, n:] == 7).all()


def _replay_us(plan, reps=50, groups=7):
    times = []
    for _ in range(groups + 1):  # the first a warm-up
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            plan.launch("graph")
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / reps)
    return min(times[1:])


def test_a_cu_per_tile_takes_as_long_as_one_tile():
    """64 graphs of 128 vertices against one: a quarter of the GPU's 256 CUs each
    close one tile.  The 256-thread closure, made to share a CU, takes 1.5
    times as long; 1.3 lies between."""
    one = torch.zeros((128, 128), device="cuda")
    many = torch.zeros((64, 128, 128), device="cuda")
    solve, batch = fw.SolvePlan(one), fw.BatchPlan([many[g] for g in range(64)])
    try:
        alone, together = _replay_us(solve), _replay_us(batch)
    finally:
        solve.destroy()
        batch.destroy()
    print(f"[batched closures] one {alone:.1f} us, 64 {together:.1f} us", flush=True)
    assert together <= 1.3 * alone


@pytest.mark.parametrize("extra", ["one", "below", "grid", "above", "twice"])
def test_persistent_counts(extra):
    """Graphs of the persistent kernel: fewer than its workgroups (each takes
    the graph of its own number), as many, and more (the rest from the counter),
    on every launch of a plan."""
    many = [torch.zeros((2, 2), device="cuda") for _ in range(8192)]
    plan = fw.BatchPlan(many)
    grid = plan.grid
    plan.destroy()
    assert 1 < grid < 8192
    count = {"one": 1, "below": grid - 1, "grid": grid, "above": grid + 1,
             "twice": 2 * grid + 3}[extra]
    rng = np.random.default_rng(count)
    sizes = rng.integers(1, 9, count)
    sizes[0] = 8
    graphs = [gen.dense_graph(int(n), 0.5, 1, 50, seed=(g, int(n))) for g, n in enumerate(sizes)]
    want = [oracle.fw(w) for w in graphs]
    src = [torch.from_numpy(w).cuda() for w in graphs]
    d = [s.clone() for s in src]
    plan = fw.BatchPlan(d)
    try:
        for mode in ("kernel", "graph", "graph"):
            for a, b in zip(d, src):
                a.copy_(b)
            plan.launch(mode)
            torch.cuda.synchronize()
            assert all(np.array_equal(a.cpu().numpy(), w) for a, w in zip(d, want)), mode
    finally:
        plan.destroy()
