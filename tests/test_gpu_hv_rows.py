"""One-pass H.v over short rows (plan down 8) against the two passes and the oracle.

Both sum every element in the same order with the same roundings, so they agree bit for bit: over row
lengths around multiples of 64 columns, row counts that are no multiple of the group, more hops than one
list holds (48 and more), sectors without hops, padded rows, and inputs with infinities and NaN.
"""
import numpy as np
import pytest

import oracle
import synth
from tests._gpu import torch_cuda, to_dev, to_host, EPS32, EPS64

pytestmark = pytest.mark.gpu


def _ring(N):
    return [(i, (i + 1) % N, 1.0 + 0.25 * (i % 3)) for i in range(N)]


def _torus(lx, ly, tp):
    return [(b.i, b.j, b.t) for b in synth.torus_nnn(lx, ly, 1.0, tp)]


CASES = [
    (8, _ring(8), 4, 4),              # 70 x 70
    (33, None, 0, 0),                 # placeholder, replaced below
    (9, _torus(3, 3, -0.3), 5, 3),    # 126 x 84
    (12, _torus(4, 3, 0.2), 6, 6),    # 924 x 924, up to 48 hops a row
    (12, _torus(4, 3, 0.0), 5, 2),    # 792 x 66
    (11, _ring(11), 3, 4),            # 165 x 330
    (13, _ring(13), 1, 4),            # 13 x 715: fewer rows than CUs
    (10, _ring(10), 0, 5),            # one row, no up hops
    (10, [], 3, 4),                   # no bonds: diagonal only
    (14, _ring(14), 6, 2),            # 3003 x 91
]
CASES[1] = (12, _ring(12), 4, 11)     # 495 x 12: too short for one pass (the plan is refused)


def _problem(args):
    import paper_1707_03974_amd as pdz
    n, bonds, nu, nd = args
    return pdz.Problem(n, bonds, 3.25, nu, nd)


def _bits(t):
    torch = torch_cuda()
    return t.view(torch.int64 if t.dtype == torch.float64 else torch.int32)


@pytest.mark.parametrize("args", CASES, ids=lambda a: f"{a[0]}s{len(a[1])}b_{a[2]}_{a[3]}")
def test_one_pass_equals_two_passes_bitwise(args):
    torch = torch_cuda()
    import paper_1707_03974_amd as pdz
    g = _problem(args)
    po = oracle.Problem(args[0], [b[0] for b in args[1]], [b[1] for b in args[1]], [b[2] for b in args[1]], 3.25,
                        args[2], args[3])
    x64 = synth.random_vector(g.D, 3)
    rows = np.unique(np.concatenate([np.random.default_rng(1).integers(0, g.D, 400), [0, g.D - 1]]))
    for name, dt, eps in (("f64", torch.float64, EPS64), ("f32", torch.float32, EPS32)):
        if g.info["D_dn"] < 33:
            assert g.get_plan(name)["down"] != 8
            with pytest.raises(pdz.PdzError):
                g.set_plan(name, 8, 0, 0, 0)
            continue
        assert g.get_plan(name)["down"] == 8
        x = to_dev(x64, dt)
        xs = to_host(x).astype(np.float64)
        inf = x.clone()
        inf[:: max(1, g.D // 7)] = float("inf")
        inf[3:: max(4, g.D // 5)] = float("nan")
        inf[5:: max(6, g.D // 4)] = -0.0
        pitch = g.info["D_dn"] + 3
        xp = torch.full((g.info["D_up"], pitch), float("nan"), dtype=dt, device="cuda")
        xp[:, :pitch - 3] = x.view(g.info["D_up"], -1)
        one, one_inf, one_p = g.hv(x), g.hv(inf), g.hv_pitched(xp.view(-1), pitch)
        g.set_plan(name, 0, 128, 1, 3)
        assert g.get_plan(name)["down"] != 8
        two, two_inf = g.hv(x), g.hv(inf)
        g.set_plan(name, 0, 0, 0, 0)
        assert torch.equal(_bits(one), _bits(two))
        assert torch.equal(one_p.view(-1, pitch)[:, :pitch - 3].reshape(-1), two)
        assert torch.equal(torch.isnan(one_inf), torch.isnan(two_inf))
        ok = ~torch.isnan(one_inf)
        assert torch.equal(one_inf[ok], two_inf[ok])
        ref, asum, nterm = oracle.hv_rows(po, xs, rows, with_abs=True)
        err = np.abs(to_host(one[torch.from_numpy(rows).cuda()]).astype(np.float64) - ref)
        assert np.all(err <= (nterm + 2) * eps * asum + nterm * EPS64 * asum)


def test_lanczos_on_one_pass_products():
    """The partial sums of q . H q that the one pass writes give the oracle's energy in both storages."""
    torch = torch_cuda()
    g = _problem(CASES[5])
    po = oracle.Problem(11, [b[0] for b in CASES[5][1]], [b[1] for b in CASES[5][1]], [b[2] for b in CASES[5][1]],
                        3.25, 3, 4)
    from scipy.sparse.linalg import eigsh
    H = oracle.build_csr(po)
    E = float(eigsh(H, k=1, which="SA", tol=1e-13, v0=np.random.default_rng(2).standard_normal(g.D))[0][0])
    for storage, tol, bound in (("f64", 1e-12, 1e-10), ("f32", 1e-7, 1e-8)):
        ya, yb = (torch.empty(g.D, dtype=torch.float64, device="cuda") for _ in range(2))
        a = g.lanczos(storage=storage, tol=tol, max_iter=400, ritz=ya)
        b = g.lanczos(storage=storage, tol=tol, max_iter=400, ritz=yb, keep_basis=1, use_graph=0)
        assert abs(a["E0_refined"] - E) <= bound * abs(E)
        assert a["E0"] == b["E0"] and torch.equal(ya, yb)     # kept and regenerated vectors, graph and stream


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_alpha_from_more_partial_sums_than_one_work_group_adds(storage):
    """92,378 rows give 23,095 partial sums of q . H q: alpha and beta of the first steps against plain dot
    products of the same vectors (FP64; rounding of 1.6e7 terms in any order, below 1e-12)."""
    torch = torch_cuda()
    dt = torch.float64 if storage == "f64" else torch.float32
    g = _problem((19, _ring(19), 9, 2))
    v = to_dev(synth.random_vector(g.D, 8), dt)
    r = g.lanczos(v0=v, storage=storage, max_iter=3, tol=0.0, coefficients=True)
    q, hq = v.double(), g.hv(v).double()
    n2 = (q @ q).item()
    a0 = (q @ hq).item() / n2
    assert abs(r["alpha"][0] - a0) <= 1e-12 * abs(a0)
    w = hq - a0 * q
    b1 = (w.norm() / n2 ** 0.5).item()
    assert abs(r["beta"][1] - b1) <= (1e-12 if storage == "f64" else 1e-6) * b1
