"""Pivoted panels at their edges: the last panel of 30 (N = 30: fewer rows than a
panel has columns, one node), 24, 14, 14 and 30 columns (N = 120, 270, 750, 1470), one and
two levels of the pivot tournament.  An LU solve with partial pivoting leaves
|Z X - B| <= c n u |Z| |X| with a modest growth factor: 1e-13 in FP64; mixed
levels refine to 1e-10 and get 1e-9."""

import ctypes as C

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_pivoted_panels(nu, precision):
    import torch
    from paper_2308_01457_amd import fosb
    ctx = fosb.Context(0)
    m = fosb.Mesh(ctx, *workloads.ellipsoid(nu, (0.7, 1.0, 1.3)))
    Z = fosb.assemble(ctx, m, 1.5)
    A = Z.cpu().numpy()
    fp64 = precision == "fp64"
    lv = fosb.Level(ctx, m, 1.5, Z, fosb.FP64 if fp64 else fosb.MIXED)
    B = np.random.default_rng(nu).standard_normal((A.shape[0], 3, 2)) @ np.array([1.0, 1j])
    for M, solve in ((A, lv.solve), (A.conj().T, lv.solve_adjoint)):
        X = torch.from_numpy(B.copy()).to(ctx.torch_device)
        solve(X)
        x = X.cpu().numpy()
        res = np.linalg.norm(M @ x - B, axis=0) / (np.linalg.norm(A) * np.linalg.norm(x, axis=0))
        assert res.max() < (1e-13 if fp64 else 1e-9)


@pytest.mark.parametrize("nrhs", [1, 5, 70])
def test_fp64_leaf_inverses(nrhs):
    """FP64 solves through 256-row leaf inverses (from N = 2048 on; N = 2430 ends in a
    block of 126 rows), forward and adjoint, in place in a wider array: the bound
    above, and the columns beside the right-hand sides untouched."""
    import torch
    from paper_2308_01457_amd import fosb
    ctx = fosb.Context(0)
    m = fosb.Mesh(ctx, *workloads.ellipsoid(9, (0.7, 1.0, 1.3)))
    Z = fosb.assemble(ctx, m, 1.5)
    A = Z.clone()
    lv = fosb.Level(ctx, m, 1.5, Z, fosb.FP64)
    for adjoint in (False, True):
        g = torch.Generator().manual_seed(nrhs)
        W = torch.randn((A.shape[0], nrhs + 3), dtype=torch.complex128, generator=g).to(ctx.torch_device)
        B = W[:, :nrhs].clone()
        rest = W[:, nrhs:].clone()
        call = fosb.lib().fosb_level_solve_adjoint if adjoint else fosb.lib().fosb_level_solve
        fosb._check(call(ctx.h, lv.h, C.c_void_p(W.data_ptr()), nrhs + 3, nrhs, C.byref(fosb.Stats())))
        X = W[:, :nrhs]
        R = torch.matmul(A.mH.contiguous() if adjoint else A, X.contiguous()) - B
        assert float((R.norm(dim=0) / (A.norm() * X.norm(dim=0))).max()) < 1e-13
        assert torch.equal(W[:, nrhs:], rest)
