"""Reachability's bulk on the matrix cores (every call outside a capture) and
on the vector units (under capture): the edges of the row tiles (32), of the
256-vertex blocks and of the 32-word strips, word counts that end inside a
wave's 8 words, and padded row strides. Whole results against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd.gen import dense_graph

pytestmark = pytest.mark.gpu

SIZES = [257, 258, 287, 289, 320, 511, 513, 544, 767, 769, 1023, 1057, 1281]


def _graph(n, seed):
    p = 1.5 / n if seed % 2 else 4.0 / n
    w = dense_graph(n, p, 1, 1, seed=(n, seed), dtype=np.int32)
    return (w == 1).astype(np.int32)


def _want(adj):
    m = adj.copy()
    np.fill_diagonal(m, 1)
    return oracle.fw_maxmin(m)


def _packed(adj, pad):
    n = adj.shape[0]
    words = fw.words_per_row(n)
    whole = torch.full((n, words + pad), 0x55555555, dtype=torch.int32, device="cuda")
    view = whole[:, :words]
    view.copy_(fw.pack_bits(torch.from_numpy(adj).cuda()))
    return view, whole, words


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("pad", [0, 1, 3])
def test_eager(n, pad):
    adj = _graph(n, pad)
    view, whole, words = _packed(adj, pad)
    fw.fw_transitive_closure_bits(view, n)
    got = fw.unpack_bits(view.contiguous(), n).cpu().numpy()
    assert np.array_equal(got, _want(adj))
    assert (whole[:, words:] == 0x55555555).all()


@pytest.mark.parametrize("n", [300, 513])
def test_captured(n):
    adj = _graph(n, 1)
    src, _, _ = _packed(adj, 0)
    bits = src.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        fw.fw_transitive_closure_bits(bits, n, stream=torch.cuda.current_stream())
    want = _want(adj)
    for _ in range(3):
        bits.copy_(src)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(fw.unpack_bits(bits, n).cpu().numpy(), want)
