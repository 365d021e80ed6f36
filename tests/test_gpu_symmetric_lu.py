"""The symmetric FP32 factorisation of MIXED EFIE levels (no pivoting, trailing
updates of the lower triangle only, fosb_opts.lu_pivoting = 0), on the s = 4
sphere of the mixed_k5 workload (N = 7680, k = 5):

* it is the factorisation kept for the Galerkin EFIE matrix (complex
  symmetric: G and the RWG pairing are symmetric in the two arguments), and its
  refined solves and first moments agree with those of the pivoted FP32
  factorisation (lu_pivoting = 1) and of the FP64 level;
* a matrix that is not symmetric, or whose leading pivot vanishes, or whose
  elimination without pivoting grows the entries past the 1e3 limit, falls back to
  partial pivoting, and the refined solves still meet the FP64 residual bound
  for that matrix."""

import pytest

import workloads

pytestmark = pytest.mark.gpu

IR_TOL = 1e-12


@pytest.fixture(scope="module")
def fz():
    import torch
    from paper_2308_01457_amd import fosb
    assert torch.cuda.is_available()
    ctx = fosb.Context(0)
    w = workloads.workload("mixed_k5")
    V, F = w.meshes[w.levels.index(4)]
    m = fosb.Mesh(ctx, V, F)
    Z = fosb.assemble(ctx, m, w.k)
    print(f"[gpu] symmetric LU: s=4 sphere, N={m.n_edges}, k={w.k}", flush=True)
    return fosb, ctx, torch, w, m, Z


def _opts(fosb, piv):
    return fosb.opts_default(ir_tol=IR_TOL, ir_max_sweeps=30, lu_pivoting=piv)


def _rhs(torch, ctx, n, nrhs=4, seed=5):
    g = torch.Generator(device="cpu").manual_seed(seed)
    B = torch.randn((n, nrhs), dtype=torch.complex128, generator=g)
    return B.to(ctx.torch_device)


def _residual(torch, Z, X, B):
    """||Z X - B||_F / (||Z||_F ||X||_F) in complex128."""
    R = torch.matmul(Z, X) - B
    return float(R.norm() / (Z.norm() * X.norm()))


def test_symmetric_factorisation_matches_pivoted_and_fp64(fz):
    fosb, ctx, torch, w, m, Z = fz
    n = m.n_edges
    lv = {}
    for name, piv in (("sym", 0), ("piv", 1)):
        lv[name] = fosb.Level(ctx, m, w.k, Z, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, piv))
    Z64 = Z.clone()
    lv["fp64"] = fosb.Level(ctx, m, w.k, Z64, fosb.FP64, w.dirs, w.pols, "radial", _opts(fosb, 0))
    assert lv["sym"].factorization() == fosb.FACTOR_SYM
    assert lv["piv"].factorization() == fosb.FACTOR_LU
    assert lv["fp64"].factorization() == fosb.FACTOR_LU
    B = _rhs(torch, ctx, n)
    X, sweeps = {}, {}
    for name, l in lv.items():
        st = fosb.Stats()
        X[name] = l.solve(B.clone(), st)
        sweeps[name] = st.ir_sweeps
    rel = {name: float((X[name] - X["fp64"]).norm() / X["fp64"].norm()) for name in ("sym", "piv")}
    res = {name: _residual(torch, Z, X[name], B) for name in X}
    print(f"[gpu]   refinement sweeps {sweeps}, vs FP64 {rel}, residuals {res}", flush=True)
    assert rel["sym"] < 1e-10 and rel["piv"] < 1e-10
    assert res["sym"] < 1e-13 and res["piv"] < 1e-13
    # the FP32 factors are about as good: at most one more sweep to the same tolerance
    assert sweeps["sym"] <= sweeps["piv"] + 1
    for d in range(len(w.dirs)):
        u = {name: lv[name].first_moment(d) for name in lv}
        e = float((u["sym"] - u["fp64"]).norm() / u["fp64"].norm())
        assert e < 1e-10, (d, e)
    for l in lv.values():
        l.close()


def _perturbed_level(fosb, ctx, torch, w, m, Zp):
    lv = fosb.Level(ctx, m, w.k, Zp, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, 0))
    B = _rhs(torch, ctx, m.n_edges, seed=7)
    X = lv.solve(B.clone())
    res = _residual(torch, Zp, X, B)
    kind = lv.factorization()
    lv.close()
    return kind, res


def test_fallback_on_asymmetry(fz):
    fosb, ctx, torch, w, m, Z = fz
    Zp = Z.clone()
    zmax = float(Z.abs().max())
    Zp[0, 1] += 1e-3 * zmax      # defect 1e-3 max|Z|, above the 1e-5 limit
    kind, res = _perturbed_level(fosb, ctx, torch, w, m, Zp)
    print(f"[gpu]   asymmetric: factorisation {kind}, residual {res:.2e}", flush=True)
    assert kind == fosb.FACTOR_LU and res < 1e-13


def test_fallback_on_zero_pivot(fz):
    fosb, ctx, torch, w, m, Z = fz
    Zp = Z.clone()
    Zp[0, 0] = 0.0               # still symmetric; the first pivot vanishes exactly
    kind, res = _perturbed_level(fosb, ctx, torch, w, m, Zp)
    print(f"[gpu]   zero pivot: factorisation {kind}, residual {res:.2e}", flush=True)
    assert kind == fosb.FACTOR_LU and res < 1e-13


def test_fallback_on_growth(fz):
    fosb, ctx, torch, w, m, Z = fz
    Zp = Z.clone()
    zmax = float(Z.abs().max())
    Zp[0, 0] = 1e-7 * zmax       # tiny leading pivot, with a coupling of max|Z| to unknown 1
    Zp[0, 1] = zmax
    Zp[1, 0] = zmax              # still symmetric
    # row 1 of U is final after the first elimination step: U11 = Z11 - Z10 Z01 / Z00
    u11 = complex(Zp[1, 1] - Zp[1, 0] * Zp[0, 1] / Zp[0, 0])
    growth_bound = abs(u11) / float(Zp.abs().max())
    assert growth_bound > 1e4
    kind, res = _perturbed_level(fosb, ctx, torch, w, m, Zp)
    print(f"[gpu]   growth >= {growth_bound:.1e}: factorisation {kind}, residual {res:.2e}", flush=True)
    assert kind == fosb.FACTOR_LU and res < 1e-13


def test_narrow_solves_match_wide_solves(fz):
    """Refined solves with 1..4 right-hand sides apply the factors' blocks as
    matrix-vector products (the narrow kernel); with 5 as GEMMs.  Both meet the
    same refinement tolerance, so the same columns agree to it, and each has an
    FP64-level residual."""
    fosb, ctx, torch, w, m, Z = fz
    lv = fosb.Level(ctx, m, w.k, Z, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, 0))
    B = _rhs(torch, ctx, m.n_edges, nrhs=5, seed=11)
    wide = lv.solve(B.clone())
    for k in (1, 2, 3, 4):
        narrow = lv.solve(B[:, :k].contiguous().clone())
        rel = float((narrow - wide[:, :k]).norm() / wide[:, :k].norm())
        res = _residual(torch, Z, narrow, B[:, :k].contiguous())
        print(f"[gpu]   {k} right-hand sides: vs the 5-column solve {rel:.2e}, residual {res:.2e}", flush=True)
        assert rel < 1e-10 and res < 1e-13
    lv.close()


@pytest.mark.parametrize("nu", [9, 10, 13])
def test_symmetric_blocks_and_split_products(fz, nu):
    """The 128-column diagonal blocks and the split products at sizes that are no
    multiple of the block widths (N = 2430 = 3 * 768 + 126, 3000 = 3 * 768 + 696,
    5070 = 6 * 768 + 462), on a complex symmetric matrix whose rows and columns
    are scaled by powers of two between 2^-20 and 2^20 (S A S with A dominant on
    the diagonal).  The factors are read back from Zlow: in the unscaled norm
    ||A - L U||_F <= N 2^-24 ||L||_F ||U||_F, the rounding bound of an FP32
    elimination of that size, and the refined solve meets the FP64 residual."""
    fosb, ctx, torch, w, m_, Z_ = fz
    V, F = workloads.geodesic_sphere(nu)
    m = fosb.Mesh(ctx, V, F)
    n = m.n_edges
    print(f"[gpu] symmetric blocks: N={n}", flush=True)
    g = torch.Generator(device="cpu").manual_seed(nu)
    A = torch.randn((n, n), dtype=torch.complex128, generator=g).to(ctx.torch_device)
    A = (A + A.T) / n ** 0.5 + 4.0 * torch.eye(n, dtype=torch.complex128, device=ctx.torch_device)
    s = torch.exp2(torch.randint(-20, 21, (n,), generator=g).double()).to(ctx.torch_device)
    Z = (s[:, None] * A * s[None, :]).contiguous()
    Zlow = torch.empty((n, n), dtype=torch.complex64, device=ctx.torch_device)
    lv = fosb.Level(ctx, m, 1.0, Z, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, 0), Zlow=Zlow)
    assert lv.factorization() == fosb.FACTOR_SYM
    LU = Zlow.to(torch.complex128) / s[:, None] / s[None, :]      # L and U of A up to S: (S L S^-1)(S U S)
    U = torch.triu(LU)
    Lf = torch.tril(Zlow.to(torch.complex128) / s[:, None] * s[None, :], -1)
    Lf += torch.eye(n, dtype=torch.complex128, device=ctx.torch_device)
    err = float((A - torch.matmul(Lf, U)).norm() / (Lf.norm() * U.norm()))
    print(f"[gpu]   ||A - LU|| / (||L|| ||U||) = {err:.2e} (bound {n * 2.0 ** -24:.2e})", flush=True)
    assert err <= n * 2.0 ** -24
    B = _rhs(torch, ctx, n, nrhs=3)
    X = B.clone()
    lv.solve(X)
    assert _residual(torch, Z, X, B) < 1e-13


@pytest.mark.parametrize("nrhs", [255, 256, 300])
def test_split_products_in_wide_solves(fz, nrhs):
    """Refined solves on both sides of the width at which the triangular solves'
    coupling products turn to the split form (256 columns; 300 ends inside a tile),
    forward and adjoint, with right-hand sides of magnitudes 1e-12 .. 1e12 by
    column: the FP64 residual bound of every column."""
    fosb, ctx, torch, w, m, Z = fz
    n = m.n_edges
    lv = fosb.Level(ctx, m, w.k, Z, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, 0))
    B = _rhs(torch, ctx, n, nrhs=nrhs, seed=nrhs)
    B = B * torch.logspace(-12, 12, nrhs, dtype=torch.float64, device=B.device)[None, :]
    zn = Z.norm()
    for adjoint in (False, True):
        X = B.clone()
        if adjoint:
            lv.solve_adjoint(X)
        else:
            lv.solve(X)
        R = torch.matmul(Z.mH.contiguous() if adjoint else Z, X) - B
        worst = float((R.norm(dim=0) / (zn * X.norm(dim=0))).max())
        print(f"[gpu]   {nrhs} columns, adjoint {adjoint}: worst column residual {worst:.1e}", flush=True)
        assert worst < 1e-9   # refinement stops by the whole block's norm: small columns carry the FP32 solve's accuracy


@pytest.mark.parametrize("nrhs", [1, 5, 65])
def test_adjoint_solves_of_symmetric_levels(fz, nrhs):
    """Adjoint solves through the conjugated forward factors, with the EFIE matrix
    and with the sign-symmetrised PMCHWT one: |Z^H X - B| <= 1e-9 |Z| |X| by column
    (refinement stops at a relative correction of 1e-10)."""
    fosb, ctx, torch, w, m, Z = fz
    levels = [(Z, fosb.Level(ctx, m, w.k, Z, fosb.MIXED, w.dirs, w.pols, "radial", _opts(fosb, 0)))]
    V, F = workloads.icosphere(3)
    mp = fosb.Mesh(ctx, V, F)   # 2N = 3840
    Zp = fosb.assemble_pmchwt(ctx, mp, w.k, 2.1)
    levels.append((Zp, fosb.Level.pmchwt(ctx, mp, w.k, 2.1, 1.0, Zp, fosb.MIXED, w.dirs, w.pols)))
    for A, lv in levels:
        assert lv.factorization() == levels[0][1].factorization()
        B = _rhs(torch, ctx, A.shape[0], nrhs=nrhs, seed=nrhs)
        X = B.clone()
        lv.solve_adjoint(X)
        R = torch.matmul(A.mH.contiguous(), X) - B
        assert float((R.norm(dim=0) / (A.norm() * X.norm(dim=0))).max()) < 1e-9


@pytest.mark.parametrize("nu, pivoting", [(8, 0), (9, 0), (9, 1), (10, 0), (11, 1)])
@pytest.mark.parametrize("nrhs", [1, 33])
def test_block_inverses_at_their_edges(nu, pivoting, nrhs):
    """Mixed solves with leaf inverses of 256 rows (N = 1920) and of 1024 rows with
    short last blocks (N = 2430: 382 rows, 3000: 952, 3630: 558), symmetric and pivoted
    factors.  Residual as in the tests above; at most three sweeps, as a wrong
    inverse would show in the contraction first (FP32 factors: 1e-4 or less a sweep)."""
    import torch
    from paper_2308_01457_amd import fosb
    ctx = fosb.Context(0)
    m = fosb.Mesh(ctx, *workloads.ellipsoid(nu, (0.8, 1.0, 1.2)))
    Z = fosb.assemble(ctx, m, 2.0)
    lv = fosb.Level(ctx, m, 2.0, Z, fosb.MIXED, opts=fosb.opts_default(lu_pivoting=pivoting))
    for adjoint in (False, True):
        B = _rhs(torch, ctx, m.n_edges, nrhs=nrhs, seed=nu)
        X, st = B.clone(), fosb.Stats()
        (lv.solve_adjoint if adjoint else lv.solve)(X, st)
        R = torch.matmul(Z.mH.contiguous() if adjoint else Z, X) - B
        assert float((R.norm(dim=0) / (Z.norm() * X.norm(dim=0))).max()) < 1e-9
        assert st.ir_sweeps <= 3
