"""First level of the dense class (blocks of up to 128 x 63 in registers) at its edges: the
row and column limits (128 / 129 rows, 63 / 64 columns), columns that outgrow it midway and
go on to the second level, blocks with more entries than its value buffer, drops in several
loops, kept factors, and values far from 1 (the Householder scalars' general path)."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare, compare_grad, run_gpu

pytestmark = pytest.mark.gpu
DROP = {"none": oracle.DROP_NONE, "fixed": oracle.DROP_FIXED, "adaptive": oracle.DROP_ADAPTIVE}


def _dense(n, density, seed):
    rng = np.random.default_rng(seed)
    d = np.where(rng.random((n, n)) < density, rng.standard_normal((n, n)), 0.0)
    np.fill_diagonal(d, 0.0)
    np.fill_diagonal(d, rng.uniform(0.6, 1.2, n) * (np.abs(d).sum(axis=0) + 0.5))
    return gen.from_dense(d)


@pytest.mark.parametrize("n,density,lmax", [(63, 1.0, 1), (64, 1.0, 1), (65, 0.9, 2), (126, 0.1, 3), (128, 0.12, 2),
                                            (129, 0.12, 2), (140, 0.08, 4), (40, 1.0, 2)])
def test_limits_on_dense_matrices(n, density, lmax):
    """Random matrices, dense (63 x 63 blocks of 3969 entries, 64 x 64 past the column limit)
    and sparser ones whose |J_k| and |I_k| pass 63 columns and 128 rows in later loops."""
    A = _dense(n, density, seed=n)
    for drop in ("fixed", "none"):
        kw = dict(c=3, lmax=lmax, eps=0.02, tol=4e-3)
        ref = oracle.rsai(A, drop=DROP[drop], **kw)
        gpu = run_gpu(A, drop=drop, **kw)
        compare(A, gpu, ref, label=f"dense-{n}-{drop}", margin_tol=1e-13)


@pytest.mark.parametrize("c,drop,N", [(1, "fixed", 21), (8, "fixed", 13), (5, "adaptive", 25), (3, "none", 19)])
def test_small_eps_grids(c, drop, N):
    """eps = 0.05 on small random-convection grids: up to lmax loops with drops in between,
    |J_k| past 63 on some columns."""
    A = gen.cd2d(N, seed=N)
    kw = dict(c=c, lmax=10 if c < 8 else 5, eps=0.05, tol=1e-3)
    ref = oracle.rsai(A, drop=DROP[drop], **kw)
    gpu = run_gpu(A, drop=drop, **kw)
    compare(A, gpu, ref, label=f"eps005-{N}-{c}-{drop}", margin_tol=1e-13)


def test_zero_diagonal_small_eps():
    """k outside I_k at the start (rows permuted): r(k) = -1 carried through the class."""
    A = gen.cd2d(14, seed=2)
    perm = np.random.default_rng(5).permutation(A.n)
    inv = np.empty(A.n, np.int64)
    inv[perm] = np.arange(A.n)
    B = gen.from_coo(A.n, inv[A.rowidx], A.col_of_entry(), A.val)
    kw = dict(c=3, lmax=10, eps=0.1, tol=1e-3)
    compare(B, run_gpu(B, drop="fixed", **kw), oracle.rsai(B, drop=oracle.DROP_FIXED, **kw), label="zero-diag-eps01",
            margin_tol=1e-13)


@pytest.mark.parametrize("scale", [1e-145, 1e-30, 1e30, 1e140])
def test_scaled_values(scale):
    """The same matrix scaled: M scales by the inverse, patterns and loops stay (no drop)."""
    A = gen.cd2d(24, seed=4)
    B = A.with_values(A.val * scale)
    kw = dict(c=3, lmax=8, eps=0.1)
    compare(B, run_gpu(B, drop="none", **kw), oracle.rsai(B, drop=oracle.DROP_NONE, **kw), label=f"scale{scale}",
            margin_tol=1e-13)


def test_kept_factors_small_eps():
    """The adjoint on factors the class kept: entry by entry against the oracle's adjoint."""
    import torch
    A = gen.cd2d(20, seed=6)
    kw = dict(c=3, lmax=8, eps=0.1, tol=1e-3)
    gpu = run_gpu(A, drop="fixed", keep_factors=True, **kw)
    assert (gpu["nJ"] > 32).sum() > 100
    g = np.random.default_rng(0).standard_normal(gpu["val"].size)
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    gpu["plan"].backward(torch.from_numpy(g).cuda(), 0.7, dA)
    want, scale = oracle.backward(A, gpu["colptr"], gpu["rowidx"], gpu["val"], g, w_frob=0.7, scale=True)
    compare_grad(dA.cpu().numpy(), want, scale, label="dense-factors")


@pytest.mark.parametrize("n", [500, 1000, 1900, 3000])
def test_tall_blocks(n):
    """Second level: blocks of 40 to 94 columns and up to 512, 1024, 2048 and more rows (the
    panel in one, two and four register rows a lane, then in memory)."""
    rng = np.random.default_rng(n)
    rows, vals = [], []
    for j in range(n):
        r = (j + 1 + rng.choice(n - 1, size=65, replace=False)) % n
        v = rng.standard_normal(65)
        rows += [j, *r]
        vals += [1.1 * np.abs(v).sum(), *v]
    A = gen.from_coo(n, rows, np.repeat(np.arange(n), 66), vals)
    kw = dict(c=1, lmax=1, eps=0.05, tol=1e-3)
    ref = oracle.rsai(A, drop=oracle.DROP_NONE, **kw)
    compare(A, run_gpu(A, drop="none", spill_capacity=n, **kw), ref, label=f"tall-{n}", margin_tol=1e-13)
