"""Chains of instances with more inputs than a lane group has lanes (nu > G >= nx): the backward
chain step's product with R~^{-1} is then too wide for the two-rows-per-load form that K' takes."""
import numpy as np
import pytest

import oracle
import treegen
from gpu_cases import TOL_GRAD, row_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nu", [(1, 15), (8, 9), (21, 43), (40, 80)])
def test_chain_with_many_inputs(nx, nu):
    import torch
    from paper_2107_01745_amd import stotree as st
    rng = np.random.default_rng([17, nx, nu])
    p = treegen.draw_problem(treegen.uniform_tree([2, 2, 1, 1]), nx, nu, rng)
    tf = st.tree_factor(p, precondition=True)
    st.sweep_schedule(tf, (8, 1, 16, 3, 16))     # a launch form that walks chains by lane groups at every size
    y = rng.standard_normal(tf.m)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda:0")   # noqa: E731
    x, u = dev(np.full(tf.x_len, np.nan)), dev(np.full(tf.u_len, np.nan))
    st.dual_grad(tf, dev(p.x0), dev(y), False, x, u)
    pb, fac = oracle.factor(p)
    xo, uo = oracle.sweep(pb, fac, row_scale(p) * y)
    s = max(1.0, np.abs(xo).max())
    assert np.abs(x.cpu().numpy() - xo.ravel()).max() / s < TOL_GRAD
    assert np.abs(u.cpu().numpy() - uo.ravel()).max() / s < TOL_GRAD
    tf.free()
