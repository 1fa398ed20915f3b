"""The fp32 canonical path behind a keyed sweep over several strips of weights
(about 2^24 weights each, so beyond 4096 vertices): scratch used strip after
strip while P gives up its weights, a ragged last strip, padded rows of both
matrices, unreachable pairs, a 64- and a 128-wide keyed sweep, a side stream, and
replays of a captured plan.  Sampled rows against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw
from paper_1001_4108_amd import gen

pytestmark = pytest.mark.gpu


def _graph(n, p, seed):
    w = gen.dense_graph(n, p, 1, 100, seed=seed, dtype=np.float32)
    w[np.isfinite(w)] += 0.25
    np.fill_diagonal(w, 0)
    return w


def _on_gpu(a, pad, fill):
    n = a.shape[0]
    whole = torch.full((n, n + pad), fill, dtype=torch.from_numpy(a[:1]).dtype, device="cuda")
    whole[:, :n] = torch.from_numpy(a)
    return whole[:, :n], whole


def _check_rows(w, d, P, rows):
    idx = torch.from_numpy(rows).cuda()
    got, hops = d[idx].cpu().numpy(), P[idx].cpu().numpy()
    want = oracle.dijkstra_rows(w, rows).astype(np.float32)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    assert np.array_equal(hops, oracle.canonical_pred(want, w, rows=rows))
    return want


# strips of 4032 columns and 68; of 3904 and 396; three, the last of 824
@pytest.mark.parametrize("n,p,tile,pad", [(4100, 0.03, 128, 0), (4300, 0.0005, 64, 1),
                                          (6200, 0.01, None, 3)])
def test_several_strips(n, p, tile, pad):
    w = _graph(n, p, n)
    d, dw = _on_gpu(w, pad, 5.0)
    P, Pw = _on_gpu(np.zeros((n, n), np.int32), pad, 5)
    before = fw.pred_fallbacks()
    if tile:
        fw.fw_apsp_plan(d, tile, pred=P)
    else:
        fw.fw_apsp_pred(d, P)
    torch.cuda.synchronize()
    assert fw.pred_fallbacks() == before + 1
    assert (dw[:, n:] == 5).all() and (Pw[:, n:] == 5).all()
    want = _check_rows(w, d, P, np.array([0, 63, 64, n // 2, n - 1]))
    assert np.isinf(want).any() == (p < 0.001)


def test_side_stream_and_plan_replays():
    n = 4225  # strips of 3968 columns and 257
    w = _graph(n, 0.02, 7)
    src = torch.from_numpy(w).cuda()
    d, P = src.clone(), torch.full((n, n), -77, dtype=torch.int32, device="cuda")
    fw.fw_apsp_pred(d, P)
    torch.cuda.synchronize()
    _check_rows(w, d, P, np.array([1, 2100, 4224]))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ds = src.clone()
        Ps = torch.full((n, n), -77, dtype=torch.int32, device="cuda")
        fw.fw_apsp_pred(ds, Ps, stream=side)
    side.synchronize()
    assert torch.equal(ds, d) and torch.equal(Ps, P)
    plan = fw.SolvePlan(ds, Ps)
    try:
        for rep in range(3):
            ds.copy_(src)
            Ps.fill_(-77)
            plan.launch("graph")
            torch.cuda.synchronize()
            assert torch.equal(ds, d) and torch.equal(Ps, P), rep
    finally:
        plan.destroy()
