"""Panel sweeps whose launches take 16 right-hand sides per workgroup (fewer than 416 nodes) and all
64 (from 416 on), on either side of that count and for every number of tasks per wavefront, against
single-vector sweeps: 1e-12 of the largest entry (sums of at most a few hundred FP64 products)."""
import numpy as np
import pytest

import treegen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nu", [(1, 1), (16, 16), (17, 3), (33, 15), (31, 33), (64, 32), (65, 63)])
@pytest.mark.parametrize("scen", [415, 416])
def test_panel_groups(nx, nu, scen):
    import torch
    from paper_2107_01745_amd import stotree as st
    rng = np.random.default_rng([23, nx, nu])
    # 1 -> 64 -> scen scenarios, then one chain stage
    p = treegen.draw_problem(treegen.capped_tree(3, scen, 64), nx, nu, rng)
    tf = st.tree_factor(p, precondition=True)
    nrhs = 64
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda:0")   # noqa: E731
    y, x0 = dev(rng.standard_normal((nrhs, tf.m))), dev(rng.uniform(-2, 2, (nrhs, nx)))
    for hom in (False, True):
        out = {}
        for n in (nrhs, 2):
            x = torch.full((nrhs, tf.x_len), np.nan, dtype=torch.float64, device="cuda:0")
            u = torch.full((nrhs, tf.u_len), np.nan, dtype=torch.float64, device="cuda:0")
            for k in range(0, nrhs, n):
                st.dual_grad(tf, x0[k:k + n], y[k:k + n], hom, x[k:k + n], u[k:k + n], nrhs=n)
            out[n] = x.cpu().numpy(), u.cpu().numpy()
        s = max(1.0, np.abs(out[2][0]).max())
        for a, b in zip(out[nrhs], out[2]):
            assert np.isfinite(a).all() and np.abs(a - b).max() <= 1e-12 * s
    tf.free()
