"""Sparse-block class on power-law columns: few, up to eight and more shared rows (closed form
and steps of the compressed solve), entry counts below and past what the lanes' registers
hold in each level, several loops with and without drops, kept factors, and the row of k
private, shared or outside the pattern."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu
DROP = {"none": oracle.DROP_NONE, "fixed": oracle.DROP_FIXED, "adaptive": oracle.DROP_ADAPTIVE}


def _both(A, drop, label, **kw):
    gpu = run_gpu(A, drop=drop, **kw)
    kw.pop("keep_factors", None)
    kw.pop("spill_capacity", None)
    compare(A, gpu, oracle.rsai(A, drop=DROP[drop], **kw), label=label, margin_tol=1e-13)


@pytest.mark.parametrize("n,maxlen,c,lmax,eps,drop", [
    (20000, 60, 3, 2, 0.1, "none"), (20000, 60, 3, 2, 0.1, "fixed"),    # 3 to 30 shared rows
    (12000, 200, 1, 3, 0.05, "none"), (12000, 200, 1, 3, 0.05, "adaptive"),  # past 1024 entries in level 0
    (12000, 400, 1, 4, 0.05, "fixed"),                                  # levels 1 to 3
    (8000, 1500, 1, 2, 0.1, "fixed"),                                   # past 4096 entries in level 3
])
def test_power_law_columns(n, maxlen, c, lmax, eps, drop):
    A = gen.powerlaw(n, seed=n, lmax=maxlen)
    _both(A, drop, f"wide-{n}-{maxlen}-{drop}", c=c, lmax=lmax, eps=eps, tol=1e-3, spill_capacity=n)


@pytest.mark.parametrize("keep", [False, True])
def test_weak_and_permuted_diagonals(keep):
    """Diagonals below the off-diagonal sums (entries of the shared rows above the private
    norms), and rows permuted (k in no column of J, in one, in several)."""
    A = gen.powerlaw(6000, seed=9, lmax=120, diag_factor=0.4)
    _both(A, "fixed", f"weak-{keep}", c=2, lmax=2, eps=0.2, tol=1e-3, spill_capacity=A.n, keep_factors=keep)
    perm = np.random.default_rng(3).permutation(A.n)
    B = gen.from_coo(A.n, perm[A.rowidx], A.col_of_entry(), A.val)
    _both(B, "fixed", f"permuted-{keep}", c=2, lmax=2, eps=0.2, tol=1e-3, spill_capacity=A.n, keep_factors=keep)
