"""Branches of the EFIE assembly against the FP64 oracle, on a stretched
icosphere.  Tolerance 1e-12 of the largest entry on the matrix: both sides
evaluate the same quadrature in FP64 (rounding of some 36 terms, phases of a
few units)."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _stretched(s):
    V, F = workloads.icosphere(s)
    return V * np.array([0.8, 1.1, 1.3]), F


@pytest.mark.parametrize("phase", [1e-3, 0.43 * (1 - 1e-9), 0.43 * (1 + 1e-9), 0.95 * (1 - 1e-9), 0.95 * (1 + 1e-9), 6.0])
def test_phase_series_at_their_limits(phase):
    """phase = 2 k h, h the largest distance of a vertex from its triangle's
    centroid: the argument bound by which the series length is chosen."""
    from oracle import efie, mesh
    from paper_2308_01457_amd import fosb
    V, F = _stretched(1)
    T = V[F]
    h = np.linalg.norm(T - T.mean(1, keepdims=True), axis=2).max()
    k = phase / (2 * h)
    ctx = fosb.Context(0)
    Z = fosb.assemble(ctx, fosb.Mesh(ctx, V, F), k).cpu().numpy()
    Zo = efie.assemble(mesh.build(V, F), k)
    assert np.abs(Z - Zo).max() / np.abs(Zo).max() < 1e-12
