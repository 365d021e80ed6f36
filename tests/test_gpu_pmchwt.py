"""Dielectric (PMCHWT) path on the GPU against the oracle (oracle/pmchwt.py)
and the Mie series:
* fosb_assemble_pmchwt: the 2N x 2N matrix entry by entry (same quadrature);
* fosb_level_create_pmchwt: first moments and the far-field map (FP64, mixed);
* the sphere experiment's rank-one second moment (fosb_correlation with
  cov = NULL, fosb_far_field_moments): CT blocks and far-field second moment
  against the oracle, and the identity Sigma_l1l2 = u_l1 u_l2^H;
* convergence of the GPU far field to the Mie series up to s = 4.
The material and incidence are the paper's sphere experiment: eps_r 2.1,
mu_r 1, k0 3, d = e_x, p = e_z, far field in the plane z = 0."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

K0, EPS, MU = 3.0, 2.1, 1.0
D, P = (1.0, 0.0, 0.0), (0.0, 0.0, 1.0)


@pytest.fixture(scope="module")
def fz():
    import torch
    from paper_2308_01457_amd import fosb
    assert torch.cuda.is_available()
    return fosb, fosb.Context(0), torch


@pytest.fixture(scope="module")
def oracle_pm():
    """Oracle PMCHWT systems (Z, b, u) and meshes at s = 1, 2."""
    from oracle import mesh as meshmod, pmchwt
    ms = {s: meshmod.build(*workloads.icosphere(s)) for s in (1, 2)}
    return ms, {s: pmchwt.solve(ms[s], K0, EPS, MU, D, P) for s in (1, 2)}


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


def _level(fosb, ctx, torch, s, precision, opts=None):
    V, F = workloads.icosphere(s)
    m = fosb.Mesh(ctx, V, F)
    Z = fosb.assemble_pmchwt(ctx, m, K0, EPS, MU)
    Zo = Z.clone() if precision == fosb.MIXED else None
    lv = fosb.Level.pmchwt(ctx, m, K0, EPS, MU, Z, precision, dirs=[D], pols=[P], opts=opts)
    return m, lv, Zo


@pytest.mark.parametrize("s", [1, 2])
def test_pmchwt_matrix_parity(fz, oracle_pm, s):
    fosb, ctx, torch = fz
    ms, sol = oracle_pm
    V, F = workloads.icosphere(s)
    m = fosb.Mesh(ctx, V, F)
    print(f"[gpu] PMCHWT assembly s={s}, 2N={2 * m.n_edges}", flush=True)
    Z = fosb.assemble_pmchwt(ctx, m, K0, EPS, MU).cpu().numpy()
    Zo = sol[s][0]
    err = np.abs(Z - Zo).max() / np.abs(Zo).max()
    print(f"[gpu]   max entry error / max entry {err:.2e}, Frobenius {_rel(Z, Zo):.2e}", flush=True)
    assert err < 1e-12


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("mixed", 1e-9)])
def test_pmchwt_level_parity(fz, oracle_pm, precision, tol):
    fosb, ctx, torch = fz
    from oracle import pmchwt
    ms, sol = oracle_pm
    prec = fosb.FP64 if precision == "fp64" else fosb.MIXED
    opts = fosb.opts_default(ir_tol=1e-12, ir_max_sweeps=20)
    m, lv, _ = _level(fosb, ctx, torch, 2, prec, opts)
    assert lv.formulation() == (fosb.FORM_PMCHWT, EPS, MU) and lv.n == 2 * m.n_edges
    u = lv.first_moment(0).cpu().numpy()
    eu = _rel(u, sol[2][2])
    xh = workloads.angles_xy(61)
    FF = fosb.far_field_matrix(ctx, lv, xh).cpu().numpy()
    FFo = pmchwt.far_field_matrix(ms[2], K0, xh).reshape(3 * 61, -1)
    ef = np.abs(FF - FFo).max() / np.abs(FFo).max()
    print(f"[gpu] PMCHWT level {precision}: first moment {eu:.2e}, far-field map {ef:.2e}", flush=True)
    assert eu < tol and ef < 1e-13


def test_pmchwt_converges_to_mie(fz):
    """GPU far field against the Mie series at s = 2, 3, 4: second order."""
    fosb, ctx, torch = fz
    from oracle import mie
    xh = workloads.angles_xy(181)
    Fm = mie.dielectric_far_field_oriented(K0, 1.0, EPS, MU, D, P, xh)
    errs = []
    for s in (2, 3, 4):
        print(f"[gpu] PMCHWT s={s} vs Mie", flush=True)
        m, lv, _ = _level(fosb, ctx, torch, s, fosb.FP64)
        u = lv.first_moment(0)
        FF = fosb.far_field_matrix(ctx, lv, xh)
        F = (FF @ u).reshape(3, -1).T.cpu().numpy()
        errs.append(_rel(F, Fm))
        lv.close()
        del FF, u
    print(f"[gpu]   errors {errs}, rates {errs[0] / errs[1]:.2f} {errs[1] / errs[2]:.2f}", flush=True)
    assert errs[2] < 4e-3 and errs[0] / errs[1] > 3.3 and errs[1] / errs[2] > 3.3


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 1e-8)])
def test_rank_one_second_moment_parity(fz, oracle_pm, precision, tol):
    """CT blocks and far-field second moment (L0 = 1, L = 2) against the oracle."""
    fosb, ctx, torch = fz
    from oracle import pmchwt
    ms, sol = oracle_pm
    prec = fosb.FP64 if precision == "fp64" else fosb.MIXED
    opts = fosb.opts_default(ir_tol=1e-12, ir_max_sweeps=20)
    xh = workloads.angles_xy(91)
    lvs = [_level(fosb, ctx, torch, s, prec, opts)[1] for s in (1, 2)]
    blocks = fosb.correlation(ctx, lvs, 1, 2, None, 0)
    var = fosb.far_field_moments(ctx, lvs, 1, 2, blocks, xh).cpu().numpy().reshape(3, -1)
    Vo, Bo, lev = pmchwt.rank_one_second_moment(ms, 1, 2, K0, EPS, MU, D, P, xh, systems=sol)
    eb = max(_rel(b.cpu().numpy(), Bo[(a, c)]) for b, (a, c, _, _) in zip(blocks, fosb.ct_pairs(1, 2)))
    ev = _rel(var, Vo)
    print(f"[gpu] rank-one CT {precision}: blocks {eb:.2e}, far-field second moment {ev:.2e}", flush=True)
    assert eb < tol and ev < tol


def test_rank_one_ct_full_ladder(fz):
    """Mixed path on s = 2..4 (2N up to 15360): every CT block is u_l1 u_l2^H
    (checked on sampled entries against the first moments), and the CT
    second moment of F_z approaches |F_z^Mie|^2."""
    fosb, ctx, torch = fz
    from oracle import mie
    xh = workloads.angles_xy(181)
    opts = fosb.opts_default(ir_tol=1e-10)
    print("[gpu] rank-one CT s=2..4 mixed", flush=True)
    lvs = [_level(fosb, ctx, torch, s, fosb.MIXED, opts) for s in (2, 3, 4)]
    levels = [x[1] for x in lvs]
    blocks = fosb.correlation(ctx, levels, 2, 4, None, 0)
    var = fosb.far_field_moments(ctx, levels, 2, 4, blocks, xh).cpu().numpy().reshape(3, -1)
    rng = np.random.default_rng(5)
    worst = 0.0
    for b, (a, c, _, _) in zip(blocks, fosb.ct_pairs(2, 4)):
        ua = levels[a - 2].first_moment(0).cpu().numpy()
        uc = levels[c - 2].first_moment(0).cpu().numpy()
        Bh = b.cpu().numpy()
        i = rng.integers(0, Bh.shape[0], 200)
        j = rng.integers(0, Bh.shape[1], 200)
        ref = ua[i] * uc[j].conj()
        worst = max(worst, np.abs(Bh[i, j] - ref).max() / (np.abs(ua).max() * np.abs(uc).max()))
    Fm = mie.dielectric_far_field_oriented(K0, 1.0, EPS, MU, D, P, xh)
    e = _rel(var[2], np.abs(Fm[:, 2]) ** 2)
    print(f"[gpu]   blocks vs u u^H {worst:.2e}, |F_z|^2 vs Mie {e:.2e}", flush=True)
    assert worst < 1e-9 and e < 0.02


# ----------------------------------------------------------------------------- DE shape derivative
SIG, ELL = 0.01, 0.5


@pytest.fixture(scope="module")
def oracle_sd():
    """Oracle shape-derivative levels (radial field) on s = 1, 2 and their CT second moment."""
    from oracle import pmchwt_sd
    lv = {s: pmchwt_sd.Level(*workloads.icosphere(s), K0, EPS, np.array(D), np.array(P), field_kind="radial")
          for s in (1, 2)}
    xh = workloads.angles_xy(91)
    V, blocks = pmchwt_sd.second_moment(lv, 1, 2, "gaussian", SIG, ELL, xh)
    return lv, xh, V, blocks


def _sd_level(fosb, ctx, torch, s, precision, field, opts=None):
    V, F = workloads.icosphere(s)
    m = fosb.Mesh(ctx, V, F)
    Z = fosb.assemble_pmchwt(ctx, m, K0, EPS, MU)
    return m, fosb.Level.pmchwt(ctx, m, K0, EPS, MU, Z, precision, dirs=[D], pols=[P], opts=opts, field=field)


@pytest.mark.parametrize("s", [1, 2])
def test_sd_weights_parity(fz, oracle_sd, s):
    """The shape-derivative weights W (2N x 6 nt) entry by entry against the oracle."""
    fosb, ctx, torch = fz
    lv_o = oracle_sd[0][s]
    print(f"[gpu] DE shape-derivative weights s={s}", flush=True)
    m, lv = _sd_level(fosb, ctx, torch, s, fosb.FP64, "radial")
    W = lv.sd_weights(0).cpu().numpy()
    err = np.abs(W - lv_o.Wgt).max() / np.abs(lv_o.Wgt).max()
    print(f"[gpu]   max entry error / max entry {err:.2e}, Frobenius {_rel(W, lv_o.Wgt):.2e}", flush=True)
    assert err < 1e-11


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 1e-8)])
def test_sd_second_moment_parity(fz, oracle_sd, precision, tol):
    """CT variance of the dielectric shape derivative (s = 1, 2, radial Gaussian
    covariance) and its Sigma blocks against the oracle."""
    fosb, ctx, torch = fz
    _, xh, Vo, Bo = oracle_sd
    prec = fosb.FP64 if precision == "fp64" else fosb.MIXED
    opts = fosb.opts_default(ir_tol=1e-12, ir_max_sweeps=20)
    lvs = [_sd_level(fosb, ctx, torch, s, prec, "radial", opts)[1] for s in (1, 2)]
    cov = fosb.make_cov("gaussian", SIG, ELL)
    blocks = fosb.correlation(ctx, lvs, 1, 2, cov, 0)
    var = fosb.far_field_moments(ctx, lvs, 1, 2, blocks, xh).cpu().numpy().reshape(3, -1)
    eb = max(_rel(b.cpu().numpy(), Bo[(a, c)]) for b, (a, c, _, _) in zip(blocks, fosb.ct_pairs(1, 2)))
    ev = _rel(var, Vo)
    print(f"[gpu] DE second moment {precision}: blocks {eb:.2e}, variance {ev:.2e}", flush=True)
    assert eb < tol and ev < tol


def test_sd_translation_and_breathing_on_the_ladder(fz):
    """GPU only, s = 2, 3, 4 (2N up to 15360), normal field: the rigid-translation
    covariance gives Var[F'_c] -> sigma^2 k0^2 |d - x|^2 |F_c|^2, and the
    constant covariance gives sigma^2 |dF_c/da|^2 (radius derivative of the Mie
    series); both approach their limits at second order."""
    fosb, ctx, torch = fz
    from oracle import mie
    xh = workloads.angles_xy(91)
    h = 1e-3
    f = lambda a: mie.dielectric_far_field_oriented(K0, a, EPS, MU, D, P, xh)
    dF = (-f(1 + 2 * h) + 8 * f(1 + h) - 8 * f(1 - h) + f(1 - 2 * h)) / (12 * h)
    et, eb = [], []
    for s in (2, 3, 4):
        print(f"[gpu] DE shape derivative s={s}", flush=True)
        m, lv = _sd_level(fosb, ctx, torch, s, fosb.FP64, "normal")
        FF = fosb.far_field_matrix(ctx, lv, xh)
        F = (FF @ lv.first_moment(0)).reshape(3, -1).cpu().numpy()
        dd = np.sum((np.array(D)[None, :] - xh) ** 2, axis=1)[None, :]
        for kind, ref, out in (("normal_dot", 0.01 ** 2 * K0 ** 2 * dd * np.abs(F) ** 2, et),
                               ("constant", 0.01 ** 2 * np.abs(dF.T) ** 2, eb)):
            blocks = fosb.correlation(ctx, [lv], s, s, fosb.make_cov(kind, 0.01, 1.0), 0)
            var = fosb.far_field_moments(ctx, [lv], s, s, blocks, xh).cpu().numpy().reshape(3, -1)
            out.append(_rel(var, ref))
            del blocks
        lv.close()
        del FF
    print(f"[gpu]   translation {et}, breathing {eb}", flush=True)
    assert et[2] < 0.01 and et[0] / et[1] > 3.0 and et[1] / et[2] > 3.0
    assert eb[2] < 0.02 and eb[0] / eb[1] > 3.0 and eb[1] / eb[2] > 3.0


def test_sd_lowrank_route(fz):
    """Dielectric shape derivative through the low-rank covariance (s = 2, 3):
    stored and streamed weights give the same factor and variance, and the
    low-rank variance matches the dense covariance route."""
    fosb, ctx, torch = fz
    xh = workloads.angles_xy(91)
    cov = fosb.make_cov("gaussian", SIG, ELL)
    print("[gpu] DE low-rank route s=2..3", flush=True)
    stored = [_sd_level(fosb, ctx, torch, s, fosb.FP64, "radial")[1] for s in (2, 3)]
    streamed = []
    for s in (2, 3):
        V, F = workloads.icosphere(s)
        m = fosb.Mesh(ctx, V, F)
        Z = fosb.assemble_pmchwt(ctx, m, K0, EPS, MU)
        streamed.append(fosb.Level.pmchwt(ctx, m, K0, EPS, MU, Z, fosb.FP64, dirs=[D], pols=[P], field="radial",
                                          streamed=True))
    ew = _rel(streamed[1].sd_weights(0).cpu().numpy(), stored[1].sd_weights(0).cpu().numpy())
    blocks = fosb.correlation(ctx, stored, 2, 3, cov, 0)
    Vd = fosb.far_field_moments(ctx, stored, 2, 3, blocks, xh).cpu().numpy()
    lr1 = fosb.LowRank(ctx, stored, cov, 4000, 1e-11)
    lr2 = fosb.LowRank(ctx, streamed, cov, 4000, 1e-11)
    V1 = lr1.far_field_moments(2, 3, xh).cpu().numpy()
    V2 = lr2.far_field_moments(2, 3, xh).cpu().numpy()
    ey = _rel(lr2.factor(1).cpu().numpy(), lr1.factor(1).cpu().numpy())
    e12, ed = _rel(V2, V1), _rel(V1, Vd)
    print(f"[gpu]   rank {lr1.rank}; streamed vs stored: weights {ew:.1e}, factor {ey:.1e}, variance {e12:.1e}; "
          f"low-rank vs dense {ed:.1e}", flush=True)
    assert ew < 1e-15 and ey < 1e-12 and e12 < 1e-12 and ed < 1e-7
    with pytest.raises(fosb.FosbError):
        fosb.correlation(ctx, streamed, 2, 3, cov, 0)
    lr1.close()
    lr2.close()


def test_pmchwt_symmetric_factorisation(fz):
    """A MIXED PMCHWT level with 2N >= 2048 (s = 3: 2N = 3840) factors S Z,
    S = diag(I, -I) on the [J; M] halves, which is symmetric, without pivoting;
    its refined solves, adjoint solves and first moment agree with the FP64
    level's and with those of the pivoted FP32 factorisation (lu_pivoting = 1)."""
    fosb, ctx, torch = fz
    V, F = workloads.icosphere(3)
    m = fosb.Mesh(ctx, V, F)
    Z = fosb.assemble_pmchwt(ctx, m, K0, EPS, MU)
    n = Z.shape[0]
    S = torch.ones(n, dtype=torch.complex128, device=Z.device)
    S[n // 2:] = -1.0
    SZ = S[:, None] * Z
    asym = float((SZ - SZ.T).abs().max() / SZ.abs().max())
    opts = lambda piv: fosb.opts_default(ir_tol=1e-12, ir_max_sweeps=30, lu_pivoting=piv)
    lv = {name: fosb.Level.pmchwt(ctx, m, K0, EPS, MU, Z, fosb.MIXED, dirs=[D], pols=[P], opts=opts(piv))
          for name, piv in (("sym", 0), ("piv", 1))}
    lv["fp64"] = fosb.Level.pmchwt(ctx, m, K0, EPS, MU, Z.clone(), fosb.FP64, dirs=[D], pols=[P])
    print(f"[gpu] PMCHWT s=3 (2N={n}): max|SZ - (SZ)^T| / max|SZ| = {asym:.2e}, factorisations "
          f"{ {k: l.factorization() for k, l in lv.items()} }", flush=True)
    assert lv["sym"].factorization() == fosb.FACTOR_SYM
    assert lv["piv"].factorization() == fosb.FACTOR_LU
    g = torch.Generator(device="cpu").manual_seed(13)
    B = torch.randn((n, 3), dtype=torch.complex128, generator=g).to(Z.device)
    for adjoint in (False, True):
        X = {}
        for name, l in lv.items():
            st = fosb.Stats()
            X[name] = (l.solve_adjoint if adjoint else l.solve)(B.clone(), st)
        for name in ("sym", "piv"):
            rel = float((X[name] - X["fp64"]).norm() / X["fp64"].norm())
            print(f"[gpu]   {'adjoint ' if adjoint else ''}solve {name} vs FP64 {rel:.2e}", flush=True)
            assert rel < 1e-10
        Zop = Z.conj().T if adjoint else Z
        res = float((Zop @ X["sym"] - B).norm() / (Z.norm() * X["sym"].norm()))
        assert res < 1e-13
    u = {name: l.first_moment(0) for name, l in lv.items()}
    assert float((u["sym"] - u["fp64"]).norm() / u["fp64"].norm()) < 1e-10
    for l in lv.values():
        l.close()


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-8)])
def test_rank_one_blocks_equal_two_sided_solves(fz, precision, tol):
    """fosb_correlation's separated rank-one blocks against the general route (C
    formed, solved on both sides) for every pair, the second of two incidences
    and a row stride beyond the block.  FP64: both are backward stable; mixed:
    both refine to ir_tol = 1e-10, times a condition number below 100."""
    fosb, ctx, torch = fz
    prec = fosb.FP64 if precision == "fp64" else fosb.MIXED
    dirs = ((1.0, 0.0, 0.0), (0.0, 0.6, 0.8))
    pols = ((0.0, 0.0, 1.0), (1.0, 0.0, 0.0))
    lvs = []
    for s in (1, 2):
        m = fosb.Mesh(ctx, *workloads.icosphere(s))
        Z = fosb.assemble_pmchwt(ctx, m, 1.3, 2.1)
        lvs.append(fosb.Level.pmchwt(ctx, m, 1.3, 2.1, 1.0, Z, prec, dirs, pols))
    pairs = fosb.ct_pairs(1, 2)
    wide = [torch.zeros((lvs[a - 1].n, lvs[b - 1].n + 5), dtype=torch.complex128, device=ctx.torch_device)
            for a, b, _, _ in pairs]
    st = fosb.Stats()
    fosb.correlation(ctx, lvs, 1, 2, None, 1, blocks=wide, stats=st)
    assert st.n_solves == len(pairs)
    for (a, b, _, _), W in zip(pairs, wide):
        C = fosb.rhs_correlation(ctx, lvs[a - 1], lvs[b - 1], None, 1)
        S = fosb.two_sided_solve(ctx, lvs[a - 1], lvs[b - 1], C)
        n2 = lvs[b - 1].n
        e = float((W[:, :n2] - S).norm() / S.norm())
        print(f"[gpu] rank-one block ({a},{b}) {precision}: separated vs two-sided {e:.1e}", flush=True)
        assert e < tol and float(W[:, n2:].abs().max()) == 0.0


def test_captured_rank_one_blocks(fz):
    """A captured fosb_correlation with rank-one data (FP64), replayed with a new level of the
    context between capture and replay: the eager blocks, and that level's own
    first moment as it was."""
    fosb, _, torch = fz
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = fosb.Context(0, stream)
        m = fosb.Mesh(ctx, *workloads.icosphere(1))

        def level():
            Z = fosb.assemble_pmchwt(ctx, m, 1.3, 2.1)
            return fosb.Level.pmchwt(ctx, m, 1.3, 2.1, 1.0, Z, fosb.FP64)

        lv = level()
        ref = fosb.correlation(ctx, [lv], 1, 1, None, 0)[0].clone()
        out = torch.zeros_like(ref)
        fosb.correlation(ctx, [lv], 1, 1, None, 0, blocks=[out])
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            fosb.correlation(ctx, [lv], 1, 1, None, 0, blocks=[out])
        others = [level() for _ in range(3)]   # their first moments have the columns' size
        u = [o.first_moment(0).clone() for o in others]
        for _ in range(3):
            out.zero_()
            graph.replay()
            stream.synchronize()
            assert torch.equal(out, ref)
            for o, v in zip(others, u):
                assert torch.equal(o.first_moment(0), v)
        for l in (lv, *others):
            l.close()
        ctx.close()
