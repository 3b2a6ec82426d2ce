"""Adjoint on kept factors over its entry counts: columns of M whose A-columns hold up to 128
entries (registers), up to 64 per lane in rounds of 64 rows (1024 entries for |J_k| <= 32,
4096 above), and more (row by row), one and several rounds."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare_grad, run_gpu

pytestmark = pytest.mark.gpu


def _circulant(n, lengths, band, seed):
    """Column j: the diagonal and rows within band of j (mod n), lengths[j % len] in all."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [], [], []
    for j in range(n):
        L = lengths[j % len(lengths)]
        off = rng.choice(2 * band, size=L - 1, replace=False) - band
        r = (j + off + (off >= 0)) % n
        v = rng.standard_normal(L - 1)
        rows += [j, *r]
        cols += [j] * L
        vals += [1.1 * np.abs(v).sum() + 0.5, *v]
    return gen.from_coo(n, rows, cols, vals)


def _extents(A, ref):
    """|J_k|, entries of the columns of J_k and |I_k| for every k."""
    L = np.diff(A.colptr)
    cols = [ref["rowidx"][ref["colptr"][k]:ref["colptr"][k + 1]] for k in range(A.n)]
    q = np.array([len(c) for c in cols])
    tot = np.array([L[c].sum() for c in cols])
    m = np.array([len(np.unique(np.concatenate([A.rowidx[A.colptr[j]:A.colptr[j + 1]] for j in c]))) for c in cols])
    return q, tot, m


@pytest.mark.parametrize("lengths,band,c,lmax,covers", [
    ((7, 8, 9), 12, 2, 2, lambda q, t, m: (q <= 32) & (t > 128) & (m <= 64)),
    ((3, 3, 60, 3), 50, 1, 1, lambda q, t, m: (q <= 32) & (t > 128) & (t <= 1024) & (m > 64)),
    ((2, 2, 2, 81), 50, 1, 1, lambda q, t, m: (q <= 32) & (t > 1024)),
    ((15, 16, 17), 60, 2, 2, lambda q, t, m: (q > 32) & (t > 128) & (t <= 4096)),
    ((90, 91), 60, 1, 1, lambda q, t, m: (q > 32) & (t > 4096)),
])
def test_entry_counts(lengths, band, c, lmax, covers):
    import torch
    A = _circulant(240, lengths, band, seed=sum(lengths))
    kw = dict(c=c, lmax=lmax, eps=0.05, tol=1e-3)
    gpu = run_gpu(A, drop="none", keep_factors=True, **kw)
    assert covers(*_extents(A, gpu)).sum() >= 8
    g = np.random.default_rng(0).standard_normal(gpu["val"].size)
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    gpu["plan"].backward(torch.from_numpy(g).cuda(), 0.7, dA)
    want, scale = oracle.backward(A, gpu["colptr"], gpu["rowidx"], gpu["val"], g, w_frob=0.7, scale=True)
    compare_grad(dA.cpu().numpy(), want, scale, label=f"entries-{lengths}")
