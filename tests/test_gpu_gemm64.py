"""FP64 GEMM tiles through the solves that use them: every tile variant forced
on every size bucket, on ragged widths (edges of 32, 64 and 96 columns) and both
operand forms.  Bound: the residual of an FP64 LU solve of a few hundred unknowns,
|Z X - B| <= 1e-13 |Z| |X| by column; the tiles accumulate in the same
order, so their results are identical."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [5, 31, 64, 97, 130])
def test_every_tile_on_ragged_widths(nrhs):
    import torch
    from paper_2308_01457_amd import fosb
    V, F = workloads.icosphere(2)
    got = []
    for variant in range(3):
        ctx = fosb.Context(0)
        fosb.autotune(ctx, 2)
        fosb.autotune_load(ctx, {(1 << 40) | (ch << 39) | (m << 26) | (n << 13) | k: variant
                                 for ch in (0, 1) for m in range(12) for n in range(12) for k in range(12)})
        mesh = fosb.Mesh(ctx, V, F)
        Z = fosb.assemble(ctx, mesh, 1.0)
        Zc = Z.cpu().numpy()
        lv = fosb.Level(ctx, mesh, 1.0, Z, fosb.FP64)
        B = np.random.default_rng(nrhs).standard_normal((Zc.shape[0], nrhs, 2)) @ np.array([1.0, 1j])
        out = []
        for A, solve in ((Zc, lv.solve), (Zc.conj().T, lv.solve_adjoint)):
            X = torch.from_numpy(B.copy()).to(ctx.torch_device)
            solve(X)
            x = X.cpu().numpy()
            res = np.linalg.norm(A @ x - B, axis=0) / (np.linalg.norm(Zc) * np.linalg.norm(x, axis=0))
            assert res.max() < 1e-13
            out.append(x)
        got.append(out)
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
