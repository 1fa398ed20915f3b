"""64-wide launches on both sides of the number of tiles (700) up to which a tile
is taken in two halves of k: 26^2 tiles and 27^2, the last one of a single
vertex, aligned and unaligned rows, every arithmetic, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd import gen

pytestmark = pytest.mark.gpu


def _padded(w, pad):
    n = w.shape[0]
    host = np.full((n, n + pad), 7, dtype=w.dtype)
    host[:, :n] = w
    t = torch.from_numpy(host).cuda()
    return t[:, :n], t


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n", [1665, 1728, 1729])
@pytest.mark.parametrize("kind", ["f32", "i32", "widest"])
def test_distances(kind, n, pad):
    w = gen.dense_graph(n, 0.05, 1, 1000, seed=(n, pad),
                        dtype=np.int32 if kind == "i32" else np.float32)
    if kind == "widest":
        w = np.where(np.isinf(w), np.float32(-np.inf), w)
    d, whole = _padded(w, pad)
    if kind == "widest":
        fw.fw_apsp_semiring(d, "maxmin")
    else:
        (fw.fw_apsp if kind == "f32" else fw.fw_apsp_i32)(d)
    want = oracle.fw_maxmin(w) if kind == "widest" else oracle.fw(w)
    assert np.array_equal(d.cpu().numpy(), want)
    assert (whole[:, n:] == 7).all()
