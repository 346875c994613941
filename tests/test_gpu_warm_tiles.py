"""The warm-start network's matrix products at the edges of their tiles (32, 64 and 128 rows and
columns, 16 rows of the reduction, 512 rows per gradient slice; the row count where the tall tiles
start) against the same products in FP64.

Tolerance: FP32 sums of K <= 512 products of values of order one carry at most a few hundred
roundings of 6e-8, below 1e-4 of the largest entry (the tolerance of the other network tests)."""
import numpy as np
import pytest

import oracle.mlp as om

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1, 1), (31, 15, 31, 32), (33, 17, 33, 33), (300, 16, 64, 64), (511, 76, 65, 65), (513, 40, 129, 31),
         (1025, 200, 160, 129), (32767, 21, 128, 30), (32768, 21, 64, 30), (32769, 20, 130, 63)]


@pytest.mark.parametrize("rows,din,dh,dout", SIZES, ids=lambda v: str(v))
def test_network_tiles(rows, din, dh, dout):
    import torch
    from paper_2107_01745_amd import stotree as st
    rng = np.random.default_rng([5, rows, din, dh, dout])
    n = om.layout(din, dh, dout)["n"]
    p = (rng.standard_normal(n) * 0.2).astype(np.float32)
    X = rng.standard_normal((rows, din)).astype(np.float32)
    dY = (rng.standard_normal((rows, dout)) / rows).astype(np.float32)
    f32 = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")   # noqa: E731
    P, Xd, dYd = f32(p), f32(X), f32(dY)
    H = torch.full((2, rows, dh), np.nan, device="cuda:0")
    Y = torch.full((rows, dout), np.nan, device="cuda:0")
    st.warm_mlp_forward(rows, din, dh, dout, P, Xd, H, Y)
    W1, b1, W2, b2, W3, b3 = om.unpack(p.astype(np.float64), din, dh, dout)
    H1 = np.maximum(X.astype(np.float64) @ W1 + b1, 0.0)
    H2 = np.maximum(H1 @ W2 + b2, 0.0)
    Yo = H2 @ W3 + b3
    Hg = H.cpu().numpy()
    for got, want in ((Hg[0], H1), (Hg[1], H2), (Y.cpu().numpy(), Yo)):
        assert np.abs(got - want).max() <= 1e-4 * max(1.0, np.abs(want).max())
    # backward with the device's own activations as gates
    G = torch.full((n,), np.nan, device="cuda:0")
    work = torch.full((st.warm_mlp_work_len(rows, din, dh, dout),), np.nan, device="cuda:0")
    st.warm_mlp_backward(rows, din, dh, dout, P, Xd, H, dYd, G, work)
    A1, A2 = Hg[0].astype(np.float64), Hg[1].astype(np.float64)
    D3 = dY.astype(np.float64)
    D2 = (D3 @ W3.T) * (A2 > 0)
    D1 = (D2 @ W2.T) * (A1 > 0)
    want = np.concatenate([a.ravel() for a in (X.astype(np.float64).T @ D1, D1.sum(0), A1.T @ D2, D2.sum(0),
                                               A2.T @ D3, D3.sum(0))])
    got = G.cpu().numpy()
    assert np.isfinite(got).all()
    k = 0
    for size in (din * dh, dh, dh * dh, dh, dh * dout, dout):
        w = want[k:k + size]
        assert np.abs(got[k:k + size] - w).max() <= 1e-4 * max(np.abs(w).max(), 1e-3 * np.abs(want).max())
        k += size
