"""Assembly of M at the edges of its tiles (256 columns per tile up to 40960 columns, 1024
beyond; 64 predecessor tiles read at a time): colptr, pattern and values against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 511, 513, 256 * 64, 256 * 64 + 1, 256 * 512, 256 * 512 + 1])
def test_assembly_tile_edges(n):
    """Random columns of 1 to 4 entries with a dominant diagonal: |J_k| varies along the
    columns and across the tile edges."""
    rng = np.random.default_rng(n)
    extra = rng.integers(0, 4, n) if n > 1 else np.zeros(1, int)
    cols = np.repeat(np.arange(n), extra)
    rows = (cols + 1 + rng.integers(0, max(min(n - 1, 40), 1), cols.size)) % n
    pairs = np.unique(np.stack([rows, cols], 1)[rows != cols], axis=0) if n > 1 else np.zeros((0, 2), int)
    rows = np.concatenate([pairs[:, 0], np.arange(n)])
    cols = np.concatenate([pairs[:, 1], np.arange(n)])
    vals = np.concatenate([rng.uniform(-1, 1, len(pairs)), rng.uniform(1.5, 3.0, n)])
    A = gen.from_coo(n, rows, cols, vals)
    kw = dict(c=3, lmax=4, eps=0.2, tol=1e-3)
    ref = oracle.rsai(A, drop=oracle.DROP_FIXED, **kw)
    gpu = run_gpu(A, drop="fixed", **kw)
    assert int(gpu["colptr"][-1]) == gpu["rowidx"].size == int(ref["colptr"][-1])
    compare(A, gpu, ref, label=f"assemble-{n}", margin_tol=1e-14)


@pytest.mark.parametrize("n", [256 * 160 - 1, 256 * 160, 256 * 160 + 1, 1024 * 64 + 1])
def test_tile_size_edges(n):
    """Where the tiles change from 256 to 1024 columns, and past one window of the latter."""
    test_assembly_tile_edges(n)
