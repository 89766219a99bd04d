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


@pytest.mark.parametrize("max_iter,tol", [(1, 0.0), (5, 0.0), (12, 0.0), (13, 0.0), (40, 1e-6), (300, 1e-12)])
def test_blocks_of_steps_stop_where_the_test_is_first_met(max_iter, tol):
    """Ritz pairs solved for a block of steps at a time: steps, energy and history do not depend on the
    block lengths, and stop at the first step that meets the test (found here from a run without one)."""
    import paper_1707_03974_amd as pdz
    torch_cuda()
    g = pdz.Problem.from_workload(synth.workload("ring8"))
    runs = [g.lanczos(max_iter=max_iter, tol=tol, check_every=ce, use_graph=ug, history=True, coefficients=True)
            for ce, ug in ((1, 1), (2, 0), (7, 1), (12, 0), (13, 1), (40, 1))]
    for r in runs[1:]:
        for k in ("E0", "iters", "resid_est", "converged", "thetas", "alpha", "beta"):
            assert r[k] == runs[0][k], (k, r[k], runs[0][k])
    full = g.lanczos(max_iter=max_iter, tol=0.0, history=True)
    n = runs[0]["iters"]
    assert runs[0]["thetas"] == full["thetas"][:n]
    assert runs[0]["resid_est"] <= tol * abs(runs[0]["E0"]) if runs[0]["converged"] and tol else n == full["iters"]


def test_invariant_subspace_in_the_middle_of_a_block():
    """A start vector with three eigencomponents closes the Krylov space after three steps; the steps the
    block still holds divide by a vanishing norm and must leave no trace."""
    import paper_1707_03974_amd as pdz
    torch = torch_cuda()
    g = pdz.Problem(4, [(0, 1, 0.0)], 2.0, 2, 2)      # diagonal H: U times the doubly occupied sites (0, 1, 2)
    v0 = torch.ones(g.D, dtype=torch.float64, device="cuda")
    r = g.lanczos(v0=v0, max_iter=50, tol=0.0, history=True, coefficients=True, refine=1)
    assert r["converged"] == 1 and r["iters"] == 3 and len(r["thetas"]) == 3
    assert abs(r["E0"]) <= 1e-13 and abs(r["E0_refined"]) <= 1e-13
    assert np.all(np.isfinite(r["alpha"])) and np.all(np.isfinite(r["beta"]))


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_results_do_not_depend_on_where_blocks_end(storage):
    """A vector of hundreds of partial sums (853,776 elements): the norm that ends a block or a run and the same
    norm in the middle of one are summed alike, alone and in a batch."""
    import paper_1707_03974_amd as pdz
    torch_cuda()
    probs = [pdz.Problem.from_workload(synth.workload(n)) for n in ("torus4x3", "ring8")]
    b = pdz.Batch(probs)
    full = probs[0].lanczos(storage=storage, max_iter=60, tol=0.0, history=True, coefficients=True)
    for m in range(1, 37):
        r = probs[0].lanczos(storage=storage, max_iter=m, tol=0.0, history=True, coefficients=True)
        for k, n in (("alpha", m), ("beta", m + 1), ("thetas", m)):
            assert r[k] == full[k][:n], (k, m)
    for tol in 10.0 ** -np.arange(1.0, 5.0, 0.125):
        runs = [probs[0].lanczos(storage=storage, tol=tol, check_every=ce, use_graph=ug) for ce, ug in ((1, 0), (40, 1))]
        res = [b.lanczos(storage=storage, tol=tol, check_every=ce, use_graph=ug)[0] for ce, ug in ((1, 0), (40, 1))]
        for x, y in ((runs[0], runs[1]), (res[0][0], res[1][0]), (res[0][1], res[1][1])):
            assert all(x[k] == y[k] for k in ("iters", "E0", "resid_est")), (tol, x, y)


@pytest.mark.parametrize("check_every,use_graph", [(1, 1), (10, 1), (10, 0), (40, 1)])
def test_runs_that_end_in_their_first_steps(check_every, use_graph):
    """From vectors near the ground state a run ends within the first, shorter blocks: same steps and values as
    the first steps of a run without a tolerance, for which the graph is made as well."""
    import paper_1707_03974_amd as pdz
    torch = torch_cuda()
    g = pdz.Problem.from_workload(synth.workload("ring8"))
    y = torch.empty(g.D, dtype=torch.float64, device="cuda")
    g.lanczos(tol=1e-13, ritz=y)
    noise = torch.from_numpy(synth.random_vector(g.D, 4)).cuda()
    for mix in (0.0, 1e-6, 1e-3, 1e-1):
        v0 = y + mix * noise
        full = g.lanczos(v0=v0, max_iter=60, tol=0.0, history=True, coefficients=True)
        for tol in (1e-1, 1e-2, 1e-4, 1e-6):
            r = g.lanczos(v0=v0, max_iter=60, tol=tol, check_every=check_every, use_graph=use_graph, history=True,
                          coefficients=True)
            n = r["iters"]
            assert r["converged"] == 1 and r["thetas"] == full["thetas"][:n] and r["resid_est"] <= tol * abs(r["E0"])
            assert r["alpha"] == full["alpha"][:n] and r["beta"] == full["beta"][:n + 1]
            if mix == 0.0:
                assert n <= 1 + (tol < 1e-5)


@pytest.mark.parametrize("max_iter", [1, 2, 3, 4, 5, 13, 14])
def test_runs_shorter_than_a_check_interval(max_iter):
    """Fewer steps than the first interval holds: the run ends with them, wherever its blocks would have."""
    import paper_1707_03974_amd as pdz
    torch_cuda()
    g = pdz.Problem.from_workload(synth.workload("ring8"))
    full = g.lanczos(max_iter=40, tol=0.0, history=True, coefficients=True)
    for ce, ug in ((1000, 0), (1000, 1), (12, 1), (1, 1)):
        r = g.lanczos(max_iter=max_iter, tol=0.0, check_every=ce, use_graph=ug, history=True, coefficients=True,
                      refine=1)
        assert r["iters"] == max_iter and r["converged"] == 0
        for k, n in (("thetas", max_iter), ("alpha", max_iter), ("beta", max_iter + 1)):
            assert r[k] == full[k][:n], (k, ce)
