"""Copies of one tree that finish apart, on every route a solve's sweeps can take: bands, lane groups
per stage and per node on handles too wide for bands, and panels with all 64 copies in a workgroup
(launches of 416 nodes and more), the latter with disturbances of each copy's own.  Each route skips
what has finished; iterations and solutions agree with the panels that sweep every copy to the end."""
import numpy as np
import pytest

import oracle
import treegen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    import torch
    from paper_2107_01745_amd import stotree
    assert torch.cuda.is_available()
    stotree.lib()
    return stotree


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _solve(st, base, X0, c, knobs, lam):
    import torch
    count = len(X0)
    tf = st.tree_factor_shared(base, count, precondition=True, c=c)
    st.sweep_schedule(tf, knobs)
    y = _t(np.zeros(tf.m))
    x = torch.zeros(tf.x_len, dtype=torch.float64, device="cuda:0")
    u = torch.zeros(tf.u_len, dtype=torch.float64, device="cuda:0")
    st.stotree_timing(True)
    rc, _ = st.nama_solve(tf, _t(X0.ravel()), y, x, u, st.make_opts(lam=lam, eps=1e-8, max_iter=3000))
    st.stotree_timing(False)
    phases = st.stotree_timing_read()
    infos = st.solve_info_batch(tf)
    assert rc == 0 and all(i["status"] == 0 and i["res_scaled_inf"] <= 1e-8 for i in infos), knobs
    tf.free()
    return x.cpu().numpy(), np.array([i["iters"] for i in infos]), {k: n for k, (_, n) in phases.items()}


def _base(nx, nu, N, scen, b0, xbox=3.0):
    rng = np.random.default_rng([57, nx, nu, scen, 0])
    return treegen.draw_problem(treegen.capped_tree(N, scen, b0), nx, nu, rng, xbox=xbox, ubox=0.3, x0_range=1.0)


def _step(base):
    pb, fac = oracle.factor(base)
    return 1.0 / (1.1 * oracle.power_iteration(pb, fac, True, 300))


def _agree(ref, got):
    s = max(1.0, np.abs(ref[0]).max())
    assert np.abs(got[0] - ref[0]).max() / s < 1e-6
    assert abs(got[1].mean() - ref[1].mean()) <= 1.0, (got[1], ref[1])


# (base sizes, launch form of the lane-group route, whether chains have launches of their own)
ROUTES = [((6, 3, 6, 9, 3), 0, True), ((6, 3, 5, 9, 3), 0, False),       # bands: with chain kernels, alone
          ((6, 3, 5, 9, 3), 2, True), ((24, 12, 5, 9, 3), 0, True), ((24, 12, 5, 9, 3), 2, True)]


@pytest.mark.parametrize("shape,form,chains", ROUTES, ids=str)
def test_lane_group_routes_skip_finished_copies(st, shape, form, chains):
    base = _base(*shape)
    rng = np.random.default_rng(23)
    X0 = rng.uniform(-1.0, 1.0, (64, base.nx)) * np.linspace(0.02, 1.0, 64)[:, None]
    lam = _step(base)
    ref = _solve(st, base, X0, None, (8, 1, 16, form, 1), lam)       # panels to the end: no phase launches
    assert ref[1].max() > ref[1].min()
    assert not any(ref[2].values()), ref[2]
    got = _solve(st, base, X0, None, (8, 1, 16, form, 65), lam)      # never panels
    assert (got[2]["bwd_chain"] > 0) == chains and got[2]["bwd_stages"] > 0, got[2]
    _agree(ref, got)
    _agree(ref, _solve(st, base, X0, None, (8, 1, 16, form, 16), lam))


def test_full_panels_skip_finished_copies(st):
    """420 chains (64 copies a workgroup) under 21 nodes (16 a workgroup), disturbances of each copy's
    own: the first 16 copies finish first, so their groups are skipped above s* while the chains'
    workgroups still carry them; 128 copies, whose first panel finishes before the second."""
    base = _base(4, 2, 4, 420, 21, xbox=10.0)      # every copy has a feasible point (the oracle's solve)
    rng = np.random.default_rng(29)
    X0 = rng.uniform(-1.0, 1.0, (128, base.nx))
    X0[:16] *= 0.02
    X0[16:64] *= 0.2
    c = 0.02 * rng.standard_normal((128, base.tree.V, base.nx)) * np.linspace(0.1, 1.0, 128)[:, None, None]
    c[:, 0] = 0.0
    lam = _step(base)
    panels = _solve(st, base, X0, c, (8, 1, 16, 0, 1), lam)
    assert panels[1][:16].max() < panels[1][64:].max()
    _agree(_solve(st, base, X0, c, (8, 1, 16, 0, 129), lam), panels)
    _agree(_solve(st, base, X0, c, (8, 1, 16, 2, 129), lam), panels)
