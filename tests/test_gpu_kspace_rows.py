"""H.v of momentum sectors over groups of rows that share a down momentum.

Sectors at the edges of that kernel against the oracle's terms, on sampled rows
with the tolerance of the other H.v tests, (n+2) eps sum|terms|: rows shorter
than a thread's columns, rows that end within them, groups of fewer rows than
the kernel takes at once, and rows of each block size it is built for.
"""
import pytest

from tests.test_gpu_kspace import _sampled_rows, _eps, _bonds
from synth.lattices import torus_nnn

pytestmark = pytest.mark.gpu

CASES = [
    # L1, L2, n_up, n_dn, K
    (4, 4, 8, 1, 0),     # one column a row
    (4, 4, 9, 2, 5),     # 7 and 8 columns
    (4, 4, 8, 3, 3),     # 35 columns
    (5, 3, 7, 5, 0),     # 200 and 201: one wave
    (5, 3, 2, 7, 1),     # 429: two waves; seven rows of each momentum
    (4, 4, 3, 8, 2),     # 800 to 810: four waves
    (6, 3, 2, 6, 4),     # 1026 to 1038: eight columns a thread
]


@pytest.mark.parametrize("dtype_name", ["f64", "f32"])
@pytest.mark.parametrize("L1,L2,nu,nd,K", CASES, ids=["%dx%d_%d+%d_K%d" % c for c in CASES])
def test_grouped_rows_match_the_oracle(L1, L2, nu, nd, K, dtype_name):
    bonds = _bonds(torus_nnn(L1, L2, 1.0, -0.3))
    _sampled_rows(L1, L2, _eps(L1, L2, bonds), 5.0, nu, nd, K, 160, 11, dtype_name)


# groups for FP64 alone (about 1,510 groups of two rows, 760 of four), for neither precision, for both
TABLES = [(5, 3, 5, 3, 2), (4, 3, 5, 4, 1), (4, 4, 5, 5, 7)]


@pytest.mark.parametrize("L1,L2,nu,nd,K", TABLES, ids=["%dx%d_%d+%d_K%d" % c for c in TABLES])
def test_each_precision_has_the_table_its_kernel_reads(L1, L2, nu, nd, K):
    bonds = _bonds(torus_nnn(L1, L2, 1.0, -0.3))
    for dtype_name in ("f32", "f64", "f32"):
        _sampled_rows(L1, L2, _eps(L1, L2, bonds), 5.0, nu, nd, K, 160, 12, dtype_name)
