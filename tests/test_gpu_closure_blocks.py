"""The diagonal closure in 8-vertex sub-blocks and the 64-wide tile staged
whole: sub-block remainders, the smallest tiles, both closing forms, the two
thread counts of the 64-wide launches, unaligned rows, every arithmetic.
Whole results against the oracle, bit for bit (integer weights)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd import gen

pytestmark = pytest.mark.gpu


def _on_gpu(w, pad):
    """A view of w with `pad` more columns per row, the padding a sentinel."""
    n = w.shape[0]
    host = np.full((n, n + pad), 7, dtype=w.dtype)
    host[:, :n] = w
    t = torch.from_numpy(host).cuda()
    return t[:, :n], t


# 2, 15 .. 17, 31 .. 33, 47 .. 49: sub-block remainders of one tile; 63 .. 65,
# 127 .. 129: one tile and the first of a second; 1536, 1537 and 1601: 23^2, 24^2
# and 25^2 bulk tiles (two halves of k per tile)
@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 112, 113, 127,
                               128, 129, 1536, 1537, 1601])
@pytest.mark.parametrize("dtype", [np.float32, np.int32])
@pytest.mark.parametrize("pad", [0, 1])
def test_distances(n, dtype, pad):
    w = gen.dense_graph(n, 0.3, 1, 1000, seed=(n, pad), dtype=dtype)
    view, whole = _on_gpu(w, pad)
    (fw.fw_apsp if dtype == np.float32 else fw.fw_apsp_i32)(view)
    want = oracle.fw(w)
    assert np.array_equal(view.cpu().numpy(), want)
    if pad:
        assert (whole[:, n:] == 7).all()


@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("n", [17, 50, 100, 200])
def test_diagonal_kept_and_batch_same_bits(n, tile):
    """A non-zero diagonal, and fractional weights: a graph alone and in a
    batch takes the same sums, whatever closes its tiles."""
    rng = np.random.default_rng((n, tile))
    w = gen.dense_graph(n, 0.4, 1, 50, seed=(n, tile))
    np.fill_diagonal(w, rng.integers(1, 200, n).astype(np.float32))
    d = torch.from_numpy(w).cuda()
    fw.fw_apsp_plan(d, tile)
    assert np.array_equal(d.cpu().numpy(), oracle.fw(w))
    f = w + rng.random((n, n), dtype=np.float32)
    alone = torch.from_numpy(f).cuda()
    batch = [torch.from_numpy(f).cuda() for _ in range(3)]
    try:
        fw.plan_set("f32", 2, 512, tile)
        fw.fw_apsp_plan(alone, tile)
        fw.fw_apsp_batched(batch)
    finally:
        fw.plan_reset()
    for b in batch:
        assert torch.equal(alone.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("n", [40, 64, 129, 700])
@pytest.mark.parametrize("dtype", [np.float32, np.int32])
def test_widest(n, dtype):
    w = gen.dense_graph(n, 0.3, 1, 1000, seed=n, dtype=dtype)
    low = np.float32(-np.inf) if dtype == np.float32 else np.int32(-2 ** 31)
    w = np.where(w == (np.inf if dtype == np.float32 else gen.I32_INF), low, w).astype(dtype)
    d = torch.from_numpy(w).cuda()
    fw.fw_apsp_semiring(d, "maxmin")
    want = oracle.fw_maxmin(w)
    assert np.array_equal(d.cpu().numpy(), want)
