"""Sparse-block class where a drop takes every column but one (values so large that no |m_j|
passes the tolerance, so each solve keeps the largest alone), and where blocks of many shared
rows are handed over to the dense class, with and without room there."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def _large(n, maxlen, seed):
    """Power-law columns, each scaled to a diagonal of 10^4 that is 2.4 to 3 times the sum of its
    other entries (a random factor, so that rows of short columns do not tie exactly): every
    |m_j| is below the tolerance and |m_k| the largest."""
    A = gen.powerlaw(n, seed=seed, lmax=maxlen, diag_factor=1.0)
    diag = A.rowidx == A.col_of_entry()
    val = A.val / A.val[diag][A.col_of_entry()]
    val[diag] = np.random.default_rng(seed).uniform(2.4, 3.0, n)
    return A.with_values(val * (1e4 / val[diag])[A.col_of_entry()])


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("n,maxlen,c,lmax,eps", [(20000, 200, 3, 4, 0.05), (6000, 60, 3, 4, 0.02), (6000, 400, 1, 6, 0.02)])
def test_no_column_passes(n, maxlen, c, lmax, eps, keep):
    A = _large(n, maxlen, seed=n + 1)
    kw = dict(c=c, lmax=lmax, eps=eps, tol=1e-3)
    ref = oracle.rsai(A, **kw)
    assert np.array_equal(ref["rowidx"], np.arange(n))
    # dropped to one column on rows past the register tiers (128 at most)
    assert ((ref["nJmax"] > 1) & (ref["nImax"] > 128)).sum() > 1000
    compare(A, run_gpu(A, drop="fixed", spill_capacity=n, keep_factors=keep, **kw), ref,
            label=f"all-dropped-{n}-{maxlen}", margin_tol=1e-13)


@pytest.mark.parametrize("keep", [False, True])
def test_hand_over_with_many_shared_rows(keep):
    """Blocks whose shared rows (a few hundred) no level of the class holds go on to the dense
    class; without room in its queue the call says so, and the next one is unaffected."""
    import paper_1503_04500_amd.rsai as rsai
    rng = np.random.default_rng(5)
    n = 400
    d = np.where(rng.random((n, n)) < 0.15, rng.standard_normal((n, n)), 0.0)
    np.fill_diagonal(d, 0.0)
    np.fill_diagonal(d, 1.1 * np.abs(d).sum(axis=0))
    A = gen.from_dense(d)
    kw = dict(c=1, lmax=1, eps=0.01)
    ref = oracle.rsai(A, drop=oracle.DROP_NONE, **kw)
    assert ref["nJmax"].max() <= 128 and ref["nImax"].min() > 256
    with pytest.raises(rsai.RSAIError, match="spill_capacity"):
        rsai.build(rsai.Matrix.from_host(A), drop="none", spill_capacity=8, keep_factors=keep, **kw).nnz()
    compare(A, run_gpu(A, drop="none", spill_capacity=n, keep_factors=keep, **kw), ref, label="many-shared",
            margin_tol=1e-13)
