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


@pytest.mark.parametrize("s, shuffled", [(2, True), (3, False), (3, True), (4, True)])
def test_bands_from_the_diagonal_on(s, shuffled):
    """One band (s = 2), two (s = 3) and many (s = 4), with triangles in mesh order
    and in random order (T+ and T- of most edges in different bands): entries
    from the corners, at random, and of edges that share a vertex (touching pairs)."""
    from oracle import efie, mesh
    from paper_2308_01457_amd import fosb
    V, F = _stretched(s)
    rng = np.random.default_rng(s)
    if shuffled:
        F = F[rng.permutation(len(F))]
    k = 3.0
    ctx = fosb.Context(0)
    Z = fosb.assemble(ctx, fosb.Mesh(ctx, V, F), k).cpu().numpy()
    m = mesh.build(V, F)
    assert Z.shape == (m.ne, m.ne)
    corners = [(a, b) for a in (0, 1, m.ne - 2, m.ne - 1) for b in (0, 1, m.ne - 2, m.ne - 1)]
    far = list(zip(rng.integers(0, m.ne, 300), rng.integers(0, m.ne, 300)))
    near = []
    for v in rng.integers(0, len(V), 40):
        e = m.tri_edge[np.nonzero((F == v).any(1))[0]].ravel()
        near += list(zip(rng.choice(e, 10), rng.choice(e, 10)))
    at = np.array(corners + far + near)
    Zo = efie.entries(m, k, at[:, 0], at[:, 1])
    assert np.abs(Z[at[:, 0], at[:, 1]] - Zo).max() / np.abs(Z).max() < 1e-12


@pytest.mark.parametrize("k", [1e-100, 1e-119, 1e-122, 1e-160])
def test_wavenumbers_without_squares(k):
    """Wavenumbers on both sides of the one below which the mesh's diameter is the
    unit of length (1e-120 over the diameter); the square of 1e-160 underflows."""
    from oracle import efie, mesh
    from paper_2308_01457_amd import fosb
    V, F = _stretched(1)
    ctx = fosb.Context(0)
    Z = fosb.assemble(ctx, fosb.Mesh(ctx, V, F), k).cpu().numpy()
    Zo = efie.assemble(mesh.build(V, F), k)
    assert np.abs(Z - Zo).max() / np.abs(Zo).max() < 1e-12
