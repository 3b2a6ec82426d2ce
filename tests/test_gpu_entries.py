"""Entries of a CSC matrix side by side (check, row pattern, transpose): column lengths around
the windows of 64 and the words of 1024 entries, empty columns, matrices around the sizes
where a wave takes 16 or 64 columns, and the malformed inputs each form must report."""
import numpy as np
import pytest

from paper_1503_04500_amd import gen

pytestmark = pytest.mark.gpu


def _matrix(n, lengths, seed):
    rng = np.random.default_rng(seed)
    L = np.resize(np.asarray(lengths), n)
    rows = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in L])
    colptr = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    return gen.CSC(n, colptr, rows.astype(np.int32), rng.standard_normal(rows.size))


@pytest.mark.parametrize("n,lengths", [
    (1, (1,)), (15, (3,)), (17, (5, 0, 2)), (300, (63, 64, 65)), (1100, (1024, 1, 0, 0, 7)), (2000, (200, 2, 2, 0, 3)),
    (65535, (5,)), (65536, (5,)), (65600, (8,)), (65601, (9, 1, 0)), (66000, (1, 300, 2, 0, 2, 2, 2, 2)),
])
def test_transpose(n, lengths):
    import paper_1503_04500_amd.rsai as rsai
    A = _matrix(n, lengths, seed=n)
    T = rsai.Matrix.from_host(A).transpose()
    order = np.lexsort((A.col_of_entry(), A.rowidx))
    assert np.array_equal(T.colptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(A.rowidx, minlength=n))]))
    assert np.array_equal(T.rowidx.cpu().numpy(), A.col_of_entry()[order])
    assert np.array_equal(T.val.cpu().numpy(), A.val[order])


@pytest.mark.parametrize("N", [40, 300])  # 16 and 64 columns a wave
@pytest.mark.parametrize("where", [0, 1, 2])
def test_malformed(N, where):
    """A row repeated, descending or out of range at a column's second, middle or last entry of
    a short and of a long column; every one is reported as a row-index error."""
    import paper_1503_04500_amd.rsai as rsai
    base = gen.cd2d(N, seed=1) if where < 2 else gen.dense_rows(N, 4, 90, seed=1)
    # a column of 70 entries in the last matrix, so that its wave takes the entries side by side
    A = base if where < 2 else gen.from_coo(base.n, np.concatenate([base.rowidx, np.arange(100, 170)]),
                                            np.concatenate([base.col_of_entry(), np.full(70, 5)]),
                                            np.ones(base.nnz + 70))
    j = 7 if where < 2 else 5
    s, e = int(A.colptr[j]), int(A.colptr[j + 1])
    for at, bad in ((s + 1, "repeat"), ((s + e) // 2, "descend"), (e - 1, "range"), (s, "negative")):
        r = A.rowidx.copy()
        r[at] = {"repeat": r[at - 1], "descend": r[at - 1] - 1, "range": A.n, "negative": -1}[bad]
        B = gen.CSC(A.n, A.colptr, r, A.val)
        with pytest.raises(rsai.RSAIError, match="flags 2"):
            rsai.build(rsai.Matrix.from_host(B), c=3, lmax=4, eps=0.4)


@pytest.mark.parametrize("n,lengths", [(1, (1,)), (63, (7, 8, 9)), (64, (0, 1, 16, 17)), (65, (3,)), (513, (200, 1, 0)),
                                       (4097, (7, 8, 0, 9))])
def test_spmv(n, lengths):
    """y = A x and A^T x: rows around the eight lanes of a group, empty ones, groups and
    workgroups that end past the last row. Error bound: the sum of |a_ij x_j| times the
    roundings of a sum of that many products."""
    import torch
    import paper_1503_04500_amd.rsai as rsai
    A = _matrix(n, [min(k, n) for k in lengths], seed=n + 1)
    x = np.random.default_rng(n).standard_normal(n)
    dA, dx = rsai.Matrix.from_host(A), torch.from_numpy(x).cuda()
    col = A.col_of_entry()
    for transpose, out, src in ((False, A.rowidx, col), (True, col, A.rowidx)):
        want, mag = np.zeros(n, np.longdouble), np.zeros(n)
        np.add.at(want, out, A.val.astype(np.longdouble) * x[src])
        np.add.at(mag, out, np.abs(A.val * x[src]))
        terms = np.bincount(out, minlength=n)
        y = rsai.spmv(dA, dx, transpose=transpose).cpu().numpy()
        assert np.all(np.abs(y - want) <= (terms + 1) * 2.0 ** -53 * mag)
