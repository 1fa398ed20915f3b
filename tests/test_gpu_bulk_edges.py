"""The 128-wide bulk's copies for rows of any alignment and for the tiles of a
partial last block: remainders of one vertex, of part of a 16-deep slice and of
all but one, every arithmetic, whole results against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd import gen

pytestmark = pytest.mark.gpu

SIZES = [129, 130, 144, 145, 255, 257, 383, 385, 513]


def _view(w, pad):
    n = w.shape[0]
    host = np.full((n, n + pad), 5, dtype=w.dtype)
    host[:, :n] = w
    t = torch.from_numpy(host).cuda()
    return t[:, :n], t


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("pad", [0, 1, 2, 3])
@pytest.mark.parametrize("dtype", [np.float32, np.int32])
def test_distances(n, pad, dtype):
    w = gen.dense_graph(n, 0.2, 1, 1000, seed=(n, pad), dtype=dtype)
    d, whole = _view(w, pad)
    fw.fw_apsp_plan(d, 128)
    assert np.array_equal(d.cpu().numpy(), oracle.fw(w))
    assert (whole[:, n:] == 5).all()


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("pad", [0, 1])
def test_widest(n, pad):
    w = gen.dense_graph(n, 0.2, 1, 1000, seed=n)
    w = np.where(np.isinf(w), np.float32(-np.inf), w)
    d, whole = _view(w, pad)
    try:
        fw.plan_set("f32", n, n, 128)
        fw.fw_apsp_semiring(d, "maxmin")
    finally:
        fw.plan_reset()
    assert np.array_equal(d.cpu().numpy(), oracle.fw_maxmin(w))
    assert (whole[:, n:] == 5).all()


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("pad", [0, 1])
def test_keyed_predecessors(n, pad):
    w = gen.reweighted_graph(n, 0.2, 1, 1000, -500, 500, seed=n).w
    d, _ = _view(w, pad)
    p, whole = _view(np.zeros((n, n), np.int32), pad)
    before = fw.pred_fallbacks()
    fw.fw_apsp_plan(d, 128, pred=p)
    want = oracle.fw(w)
    assert np.array_equal(d.cpu().numpy(), want)
    assert np.array_equal(p.cpu().numpy(), oracle.canonical_pred(want, w))
    assert (whole[:, n:] == 5).all()
    assert fw.pred_fallbacks() == before


def test_rows_further_apart_than_32_bit_offsets():
    n, ld = 130, (1 << 25) + 1
    w = gen.dense_graph(n, 0.2, 1, 1000, seed=n)
    d = torch.empty((n - 1) * ld + n, device="cuda").as_strided((n, n), (ld, 1))
    d.copy_(torch.from_numpy(w))
    fw.fw_apsp_plan(d, 128)
    assert np.array_equal(d.cpu().numpy(), oracle.fw(w))
