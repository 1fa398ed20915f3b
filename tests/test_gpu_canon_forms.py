"""The fp32 canonical path's two scans: weights whose sums are exact (the
minimum form decides), multiples of 2^-6 whose sums round, reals, and tiles of
small distances between large ones of both signs, where the minimum form may
start and have to leave.  Whatever the distances rounded to, the last hops are
exactly the definition's over those distances: the oracle evaluates it on the
device's own distances.  Sizes at the edges of the 64-wide tiles, the 32-deep
slices and the 8-deep groups, padded rows, and one of several strips."""
import numpy as np
import pytest
import torch

import oracle
import paper_1001_4108_amd as fw

pytestmark = pytest.mark.gpu


def _weights(n, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "exact":
        w = rng.integers(1, 400, (n, n)) / 4 + 0.25
    elif kind == "rounds":  # 24-bit multiples of 2^-6: sums of them lose bits
        w = rng.integers(1, 1 << 24, (n, n)) / 64
    elif kind == "mixed":  # block potentials up to 2^20 on weights of 4 to 400: no negative cycle
        pot = np.repeat(rng.integers(-(1 << 20), 1 << 20, n // 64 + 1), 64)[:n]
        w = rng.integers(256, 25600, (n, n)) / 64 + pot[:, None] - pot[None, :]
    else:
        w = rng.uniform(0.001, 1000.0, (n, n))
    w = w.astype(np.float32)
    w[rng.random((n, n)) > 0.4] = np.inf
    if kind != "mixed":
        w[0, n - 1] = 0.25  # no integer: never a keyed sweep
    else:
        w[0, 1] = 4.25  # (within a block)
    np.fill_diagonal(w, 0)
    return w


def _run(w, pad):
    n = w.shape[0]
    host = np.full((n, n + pad), 5, dtype=np.float32)
    host[:, :n] = w
    whole = torch.from_numpy(host).cuda()
    d = whole[:, :n]
    P = torch.full((n, n), -77, dtype=torch.int32, device="cuda")
    before = fw.pred_fallbacks()
    fw.fw_apsp_pred(d, P)
    torch.cuda.synchronize()
    assert fw.pred_fallbacks() == before + 1
    if pad:
        assert (whole[:, n:].cpu().numpy() == 5).all()
    return d.cpu().numpy(), P.cpu().numpy()


@pytest.mark.parametrize("kind", ["exact", "rounds", "mixed", "real"])
@pytest.mark.parametrize("n,pad", [(2, 0), (7, 1), (8, 0), (9, 3), (31, 0), (33, 2), (63, 0),
                                   (65, 1), (96, 0), (129, 3), (600, 0), (1153, 1)])
def test_last_hops_follow_the_definition(n, pad, kind):
    w = _weights(n, kind, n)
    print(f"[canon forms] n={n} pad={pad} {kind}", flush=True)
    d, P = _run(w, pad)
    assert np.array_equal(P, oracle.canonical_pred(d, w))


@pytest.mark.parametrize("kind", ["exact", "rounds", "mixed", "real"])
def test_several_strips(kind):
    n = 4225  # strips of 3968 columns and 257
    w = _weights(n, kind, n)
    rows = np.array([0, 1, 63, 64, 2100, 4223, 4224])
    print(f"[canon forms] n={n} {kind}", flush=True)
    d, P = _run(w, 0)
    assert np.array_equal(P[rows], oracle.canonical_pred(d[rows], w, rows=rows))
