"""Soft rows whose Huber threshold is so small that weight / threshold overflows: the penalty is then
the distance itself to the last bit, so a fixed number of iterations, its line-search trace included,
equals that of threshold 0 (a line search whose sums turn NaN accepts no step)."""
import numpy as np
import pytest

import pins
import treegen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["nama", "minfbe"])
@pytest.mark.parametrize("hub,scale", [(1e-310, 1.0), (5e-324, 1.0), (1e-300, 1e9)])
def test_threshold_near_the_smallest_doubles(method, hub, scale):
    import torch
    from paper_2107_01745_amd import stotree as st
    base = pins.soft_rows(pins.tight_tiny())
    wgt = np.where(np.isfinite(base.wgt), scale * base.wgt, np.inf)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")   # noqa: E731
    out = []
    for h in (0.0, hub):
        prob = treegen.with_soft_rows(base, wgt, np.full(base.m, h))
        tf = st.tree_factor(prob, precondition=True)
        lam = 1.0 / (1.1 * st.dual_lipschitz(tf))
        y, x, u = dev(np.zeros(tf.m)), dev(np.zeros(tf.x_len)), dev(np.zeros(tf.u_len))
        trace = dev(np.zeros((1, 12, st.TRACE_COLS)))
        solve = st.nama_solve if method == "nama" else st.minfbe_solve
        solve(tf, dev(prob.x0), y, x, u, st.make_opts(lam=lam, eps=0.0, max_iter=12, trace=trace))
        out.append((y.cpu().numpy(), x.cpu().numpy(), trace.cpu().numpy()))
        tf.free()
    (y0, x0, t0), (y1, x1, t1) = out
    assert np.isfinite(t1[..., :st.TRACE_PHI + 11]).all()  # the 11 trials of the default nu_max (columns past them are unused)
    assert np.array_equal(t1[..., 2], t0[..., 2])          # the accepted trial of every update
    assert np.abs(y1 - y0).max() <= 1e-9 * max(1.0, np.abs(y0).max())
    assert np.abs(x1 - x0).max() <= 1e-9 * max(1.0, np.abs(x0).max())
