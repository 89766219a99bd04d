"""H.v on the palindromic rows of parity subspaces, whose hop sources come from tables.

Rows that end just below one work group's 256 columns and just past it, hop
counts on both sides of a batch of eight, palindromic columns kept and left out
(the two parities), against the oracle's projected matrix with the tolerance of
the other parity H.v tests.
"""
import numpy as np
import pytest

from oracle import inversion as inv
from tests._gpu import torch_cuda, EPS64, EPS32
from tests.test_gpu_parity import _bound, _chain, _check_hv, _gpu, _open_rect, _oracle, _perm  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    (12, _chain(12, 1.0, 0.3), 4.0, 2, 4),                 # 255 or 240 columns
    (12, _open_rect(4, 3, 1.0, -0.25), 5.0, 2, 5),         # 396 columns, none a palindrome
    (11, _chain(11, 1.0, 0.0, periodic=True), 3.0, 3, 5),  # 236 or 226 columns, few hops
    (10, _open_rect(5, 2, 1.0, 0.2), 2.0, 4, 1),           # five columns
]


@pytest.mark.parametrize("dtype_name", ["f64", "f32"])
@pytest.mark.parametrize("P", [1, -1])
@pytest.mark.parametrize("case", CASES, ids=["chain12_2+4", "open4x3_2+5", "ring11_3+5", "open5x2_4+1"])
def test_palindromic_rows_match_the_oracle(case, P, dtype_name):
    torch = torch_cuda()
    N, bonds, U, nu, nd = case
    HP = inv.build_csr_P(_oracle(N, bonds, U, nu, nd), P)
    g = _gpu(N, bonds, U, nu, nd, P)
    dt, e = (torch.float64, EPS64) if dtype_name == "f64" else (torch.float32, EPS32)
    x = np.random.default_rng(31).uniform(-1, 1, g.D)
    if dtype_name == "f32":
        x = x.astype(np.float32).astype(np.float64)
    _check_hv(g, HP, x, dt, e, _perm(g, N, nu, nd, P)[0], (dtype_name, P))
