"""Ritz values and residuals of every Lanczos step against LAPACK on the returned coefficients.

T_k has diagonal alpha[0..k) and off-diagonal beta[1..k); the device solve evaluates its leading minors
in batches of eight steps, so orders around multiples of eight, orders past convergence (copies of the
lowest Ritz value) and entries far from one are the edges.  Bound: LAPACK's backward error k eps |T|
and the device's few ulps, together below 4 k eps |T|.
"""
import numpy as np
import pytest

import synth
from tests._gpu import torch_cuda

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


def _check(r, scale=1.0):
    a, b = np.array(r["alpha"]) / scale, np.array(r["beta"]) / scale
    n = len(a)
    assert len(r["thetas"]) == n == r["iters"]
    for k in range(1, n + 1):
        t = np.diag(a[:k]) + np.diag(b[1:k], 1) + np.diag(b[1:k], -1)
        norm = np.abs(t).sum(axis=1).max()
        e = np.linalg.eigvalsh(t)[0]
        assert abs(r["thetas"][k - 1] / scale - e) <= 4 * k * EPS * norm, (k, r["thetas"][k - 1], e)
    ev, vec = np.linalg.eigh(t)
    # the residual estimate beta_{n+1} |s_n| of the last step (absolute error of s_n: eps |T| / gap)
    gap = ev[1] - ev[0] if n > 1 else 1.0
    tol = b[n] * 16 * n * EPS * norm / max(gap, 1e-3 * norm) + 1e-3 * b[n] * abs(vec[-1, 0])
    if gap > 1e-3 * norm:
        assert abs(r["resid_est"] / scale - b[n] * abs(vec[-1, 0])) <= tol


@pytest.mark.parametrize("steps", [1, 2, 7, 8, 9, 16, 17, 18, 60, 300])
def test_ritz_values_of_every_step(steps):
    import paper_1707_03974_amd as pdz
    torch_cuda()
    g = pdz.Problem.from_workload(synth.workload("torus4x3"))
    _check(g.lanczos(max_iter=steps, tol=0.0, history=True, coefficients=True, seed=steps))


@pytest.mark.parametrize("power", [-30, 90])
def test_ritz_values_of_matrices_far_from_one(power):
    import paper_1707_03974_amd as pdz
    torch_cuda()
    w = synth.workload("ring8")
    s = 2.0 ** power
    g = pdz.Problem(8, [(b.i, b.j, b.t * s) for b in w.bonds], w.U * s, w.n_up, w.n_dn)
    _check(g.lanczos(max_iter=25, tol=0.0, history=True, coefficients=True), s)
