"""Kept factors of the dense class's first level (|J_k| of 33 to 63 columns, up to 128 rows)
for columns that end without a fresh solve: the last loop finds no new column, so the factor of
an earlier solve has to survive the residual phases after it."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare_grad, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,seed,c,eps,lmax", [(16, 1, 1, 0.05, 24), (16, 1, 3, 0.02, 20)])
def test_factor_of_an_earlier_solve(N, seed, c, eps, lmax):
    import torch
    A = gen.cd2d(N, seed=seed)
    kw = dict(c=c, eps=eps, tol=1e-3)
    ref, before = oracle.rsai(A, lmax=lmax, **kw), oracle.rsai(A, lmax=lmax - 1, **kw)
    inside = (ref["nJ"] > 32) & (ref["nJmax"] <= 63) & (ref["nImax"] <= 128)
    # no solve in the last loop, or no candidate row left before it
    late = (ref["resnorm"] > eps) & (((ref["loops"] == lmax) & (ref["nsolve"] == before["nsolve"])) | (ref["loops"] < lmax))
    assert (inside & late).sum() >= 2
    gpu = run_gpu(A, drop="fixed", keep_factors=True, lmax=lmax, **kw)
    g = np.random.default_rng(0).standard_normal(gpu["val"].size)
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    gpu["plan"].backward(torch.from_numpy(g).cuda(), 0.7, dA)
    want, scale = oracle.backward(A, gpu["colptr"], gpu["rowidx"], gpu["val"], g, w_frob=0.7, scale=True)
    compare_grad(dA.cpu().numpy(), want, scale, label=f"late-{N}-{c}")


@pytest.mark.parametrize("density,lmax", [(0.6, 12), (0.15, 30)])
def test_factor_beside_many_entries(density, lmax):
    """Rows 0..119 are held by columns 0..59 alone, so their loops run out of new columns with
    |J_k| of up to 60; the residual's values take many passes of the smaller buffer (some 4000 entries)
    or a few."""
    import torch
    rng = np.random.default_rng(7)
    n, h = 180, 60
    d = np.zeros((n, n))
    d[:2 * h, :h] = np.where(rng.random((2 * h, h)) < density, rng.standard_normal((2 * h, h)), 0.0)
    d[np.arange(h), np.arange(h)] = 4.0
    d[2 * h + np.arange(h), h + np.arange(h)] = 1.0  # the other columns hold rows 120..179
    d[2 * h + (np.arange(h) + 1) % h, h + np.arange(h)] = 0.5
    d[2 * h + np.arange(h), 2 * h + np.arange(h)] = 2.0
    A = gen.from_dense(d)
    kw = dict(c=1, eps=1e-3)
    ref = oracle.rsai(A, lmax=lmax, drop=oracle.DROP_NONE, **kw)
    before = oracle.rsai(A, lmax=lmax - 1, drop=oracle.DROP_NONE, **kw)
    late = (ref["nJ"] > 32) & (ref["nJ"] <= 63) & (ref["nI"] <= 128) & (ref["loops"] == lmax) & (ref["nsolve"] == before["nsolve"])
    assert late.sum() >= 40
    gpu = run_gpu(A, drop="none", keep_factors=True, lmax=lmax, **kw)
    g = rng.standard_normal(gpu["val"].size)
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    gpu["plan"].backward(torch.from_numpy(g).cuda(), 0.7, dA)
    want, scale = oracle.backward(A, gpu["colptr"], gpu["rowidx"], gpu["val"], g, w_frob=0.7, scale=True)
    compare_grad(dA.cpu().numpy(), want, scale, label=f"many-entries-{density}")
