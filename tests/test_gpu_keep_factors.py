"""keep_factors stores R beside the build and changes nothing in it: M, its residual norms and
its loops are the same bits with and without, in every size class."""
import numpy as np
import pytest

from paper_1503_04500_amd import gen
from tests.parity import compare_grad, run_gpu

pytestmark = pytest.mark.gpu

MATRICES = {
    "powerlaw": lambda: (gen.powerlaw(20000, seed=4, lmax=200), dict(c=3, lmax=10, eps=0.4)),
    "powerlaw-shared": lambda: (gen.powerlaw(6000, seed=9, lmax=60, diag_factor=0.4), dict(c=2, lmax=2, eps=0.1)),
    "grid2d": lambda: (gen.cd2d(40, seed=2), dict(c=3, lmax=8, eps=0.1)),
    "grid3d": lambda: (gen.cd3d(10, seed=2), dict(c=3, lmax=8, eps=0.3)),
    "dense-rows": lambda: (gen.dense_rows(48, 24, 20, seed=3), dict(c=3, lmax=3, eps=0.25)),
}


@pytest.mark.parametrize("drop", ["fixed", "none"])
@pytest.mark.parametrize("name", sorted(MATRICES))
def test_same_bits(name, drop):
    A, kw = MATRICES[name]()
    # (route 0: a column's classes follow from its own sizes; by default they come from estimates
    # that depend on the order of the row pattern, which may differ from build to build)
    kw = dict(kw, drop=drop, tol=1e-3, spill_capacity=A.n, route=0)
    if drop == "none":
        kw["lmax"] = min(kw["lmax"], 3)
    plain, kept = run_gpu(A, **kw), run_gpu(A, keep_factors=True, **kw)
    for key in ("colptr", "rowidx", "val", "resnorm", "loops", "nI", "nJ", "status"):
        assert np.array_equal(plain[key], kept[key]), f"{name}-{drop}: {key}"


@pytest.mark.parametrize("name", sorted(MATRICES))
def test_adjoint_on_the_kept_factors(name):
    """R of every column's final pattern, whatever way its solves took: entry by entry against
    the oracle's adjoint on the same pattern."""
    import torch

    import oracle
    A, kw = MATRICES[name]()
    gpu = run_gpu(A, drop="fixed", tol=1e-3, spill_capacity=A.n, keep_factors=True, **kw)
    g = np.random.default_rng(1).standard_normal(gpu["val"].size)
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    gpu["plan"].backward(torch.from_numpy(g).cuda(), 0.7, dA)
    want, scale = oracle.backward(A, gpu["colptr"], gpu["rowidx"], gpu["val"], g, w_frob=0.7, scale=True)
    compare_grad(dA.cpu().numpy(), want, scale, label=f"kept-{name}")
