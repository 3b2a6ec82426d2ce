"""BiCGStab's host loop around its chunks of six iterations: solves that end in a chunk's first,
last and middle iterations, before the first one, and with the largest iteration limit."""
import numpy as np
import pytest

import oracle
from paper_1503_04500_amd import gen
from tests.parity import run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grid():
    A = gen.cd2d(48, seed=5)
    return A, run_gpu(A, c=3, lmax=8, eps=0.4, tol=1e-3), A.matvec(np.ones(A.n))


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("maxit", [0, 1, 2, 5, 6, 7, 11, 12, 13])
def test_limit_around_the_chunks(grid, maxit, graph):
    import torch
    A, gpu, b = grid
    it_o, rel_o, x_o = oracle.bicgstab(A, b, (gpu["colptr"], gpu["rowidx"], gpu["val"]), maxit=maxit)
    x, it, rel = gpu["plan"].bicgstab(torch.from_numpy(b).cuda(), maxit=maxit, graph=graph)
    assert it == it_o == maxit + 1
    assert np.max(np.abs(x.cpu().numpy() - x_o)) <= 1e-10 * max(np.max(np.abs(x_o)), 1e-300)
    assert abs(rel - rel_o) <= 1e-8 * rel_o


@pytest.mark.parametrize("graph", [True, False])
def test_largest_limit_and_solves_in_a_row(grid, graph):
    """maxit = 2^31 - 1 converges as any other; a solve that ends at once (b = 0) and one that
    runs leave nothing behind for each other."""
    import torch
    A, gpu, b = grid
    want = None
    for _ in range(3):
        x, it, rel = gpu["plan"].bicgstab(torch.from_numpy(b).cuda(), maxit=2 ** 31 - 1, graph=graph)
        x0, it0, _ = gpu["plan"].bicgstab(torch.zeros(A.n, dtype=torch.float64, device="cuda"), graph=graph)
        assert rel < 1e-8 and it > 12 and it0 == 0 and not x0.any()
        got = (it, x.cpu().numpy().tobytes())
        assert want in (None, got)
        want = got
