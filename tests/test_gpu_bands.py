"""Sweeps of narrow trees in bands of stages against the CPU oracle, at the sizes where a band
can go wrong: lane groups of 8 and 16 (widths at both ends of each) and the first width past
them, one to several register batches of rows, stages with one node more or fewer than a workgroup has wavefronts,
a node with as many children as a band takes and with one more (which runs per stage),
chains inside and below the bands, and trees of several bands."""
import numpy as np
import pytest

import oracle
import treegen
from gpu_cases import TOL_GRAD, row_scale

pytestmark = pytest.mark.gpu

# (nx, nu, N, scenarios, b0)
SHAPES = [(1, 1, 3, 4, 2), (9, 7, 4, 16, 2), (8, 8, 5, 9, 3), (15, 1, 4, 8, 2), (1, 15, 4, 8, 2),   # groups of 8
          (10, 7, 4, 9, 3), (17, 15, 5, 20, 2), (31, 1, 4, 8, 2), (5, 27, 3, 6, 3),                 # groups of 16
          (20, 13, 6, 30, 3), (40, 24, 4, 12, 2), (63, 1, 3, 4, 2), (21, 43, 3, 4, 2),              # too wide for a band
          (4, 2, 9, 512, 2), (6, 3, 7, 300, 7), (3, 2, 4, 2100, 13),                                # several bands
          (5, 3, 3, 64, 64), (5, 3, 3, 65, 65), (20, 11, 3, 40, 40), (20, 11, 3, 41, 41)]         # wide fan-outs


@pytest.fixture(scope="module")
def st():
    import torch
    from paper_2107_01745_amd import stotree
    assert torch.cuda.is_available()
    stotree.lib()
    return stotree


def _prob(shape, seed=0):
    nx, nu, N, S, b0 = shape
    rng = np.random.default_rng([91, nx, nu, S, seed])
    return treegen.draw_problem(treegen.capped_tree(N, S, b0), nx, nu, rng, cross_terms=True)


def _check(st, probs, tf, nrhs, homogeneous, seed):
    import torch
    rng = np.random.default_rng(seed)
    y, x0 = rng.standard_normal((nrhs, tf.m)), rng.standard_normal((nrhs, tf.x0_len))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda:0")   # noqa: E731
    x = torch.full((nrhs, tf.x_len), np.nan, dtype=torch.float64, device="cuda:0")
    u = torch.full((nrhs, tf.u_len), np.nan, dtype=torch.float64, device="cuda:0")
    st.dual_grad(tf, dev(x0), dev(y), homogeneous, x, u, nrhs=nrhs)
    x, u = x.cpu().numpy(), u.cpu().numpy()
    for p, d in zip(probs, tf.instances):
        pb, fac = oracle.factor(p)
        for k in range(nrhs):
            xo, uo = oracle.sweep(pb, fac, row_scale(p) * y[k, d["y_off"]:d["y_off"] + d["m"]],
                                  homogeneous=homogeneous, x0=x0[k, d["x0_off"]:d["x0_off"] + d["nx"]])
            s = max(1.0, np.abs(xo).max())
            assert np.abs(x[k, d["x_off"]:d["x_off"] + xo.size] - xo.ravel()).max() / s < TOL_GRAD
            assert np.abs(u[k, d["u_off"]:d["u_off"] + uo.size] - uo.ravel()).max() / s < TOL_GRAD


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_band_sweeps(st, shape):
    p = _prob(shape)
    tf = st.tree_factor(p, precondition=True)
    for nrhs, hom in ((1, False), (2, False), (2, True)):
        _check(st, [p], tf, nrhs, hom, 5)
    tf.free()


@pytest.mark.parametrize("mode", [0, 2])
def test_band_forest(st, mode):
    """Trees of both lane-group widths in one handle; with one too wide and one too bushy for a
    band, every tree of the handle runs per stage."""
    banded = [_prob(s) for s in SHAPES if s[0] + s[1] <= 32 and s[3] < 500]
    for probs in (banded, [_prob(s) for s in SHAPES] + [_prob((50, 20, 4, 8, 2))]):
        tf = st.tree_factor_batch(probs, precondition=True)
        st.sweep_schedule(tf, (8, 1, 16, mode, 16))
        for nrhs, hom in ((1, False), (2, True)):
            _check(st, probs, tf, nrhs, hom, 7)
        tf.free()
