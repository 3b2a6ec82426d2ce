"""Register tiers on columns around a lane group's width (8 and 16 entries): the kept local
rows hold a column's first group of entries, the rest takes the looked-up path."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def _banded(n, lengths, seed):
    """Column j: the diagonal and rows near j, lengths[j % len(lengths)] entries in all."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [], [], []
    for j in range(n):
        L = lengths[j % len(lengths)]
        near = [i for i in range(max(0, j - 40), min(n, j + 41)) if i != j]
        r = rng.choice(near, size=L - 1, replace=False)
        v = rng.standard_normal(L - 1)
        rows += [j, *r]
        cols += [j] * L
        vals += [1.1 * np.abs(v).sum() + 0.5, *v]
    return gen.from_coo(n, rows, cols, vals)


@pytest.mark.parametrize("lengths", [(7, 8, 9), (1, 8, 16), (15, 16, 17), (2, 3, 24, 25), (3, 4, 33)])
@pytest.mark.parametrize("drop", ["none", "fixed"])
def test_column_lengths(lengths, drop):
    A = _banded(257, lengths, seed=sum(lengths))
    kw = dict(c=2, lmax=4, eps=0.15, tol=2e-3)
    ref = oracle.rsai(A, drop={"none": oracle.DROP_NONE, "fixed": oracle.DROP_FIXED}[drop], **kw)
    compare(A, run_gpu(A, drop=drop, **kw), ref, label=f"columns-{lengths}-{drop}", margin_tol=1e-13)
