"""Wide mixed solves, whose coupling products run on the fp16 matrix cores: from 256
columns and 256 of K on, once the 256 x 128 tiles cover half of the compute
units.  At N = 7680 the largest coupling has 4096 rows (symmetric factors, leaves of
1024) or 3840 (the pivoted adjoint, leaves of 256), so 1100 columns, which end
inside a tile, are enough."""

import pytest

import workloads

pytestmark = pytest.mark.gpu

NRHS = 1100


@pytest.fixture(scope="module")
def fz():
    import torch
    from paper_2308_01457_amd import fosb
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert (3840 // 256) * -(-NRHS // 128) >= cu // 2
    ctx = fosb.Context(0)
    return fosb, ctx, torch, fosb.Mesh(ctx, *workloads.geodesic_sphere(16))


def _rhs(torch, dev, n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn((n, NRHS), dtype=torch.complex128, generator=g).to(dev)


def _solve(lv, adjoint, B):
    X = B.clone()
    (lv.solve_adjoint if adjoint else lv.solve)(X)
    return X


@pytest.mark.parametrize("pivoting", [0, 1])
def test_columns_of_any_magnitude(fz, pivoting):
    """Right-hand sides of magnitudes 1e-12 .. 1e12 by column, with the EFIE matrix:
    |Z X - B| <= 1e-9 |Z| |X| by column."""
    fosb, ctx, torch, m = fz
    Z = fosb.assemble(ctx, m, 2.0)
    lv = fosb.Level(ctx, m, 2.0, Z, fosb.MIXED, opts=fosb.opts_default(lu_pivoting=pivoting, ir_tol=1e-12))
    B = _rhs(torch, Z.device, m.n_edges, 1)
    B = B * torch.logspace(-12, 12, NRHS, dtype=torch.float64, device=B.device)[None, :]
    for adjoint in (False, True):
        X = _solve(lv, adjoint, B)
        R = torch.matmul(Z.mH.contiguous() if adjoint else Z, X) - B
        worst = float((R.norm(dim=0) / (Z.norm() * X.norm(dim=0))).max())
        print(f"[gpu] {NRHS} columns, pivoting {pivoting}, adjoint {adjoint}: residual {worst:.1e}", flush=True)
        assert worst < 1e-9
    lv.close()


@pytest.mark.parametrize("pivoting", [0, 1])
def test_unused_rows_take_no_bits(fz, pivoting):
    """Z = diag(A, 1e-15 I): the last 2048 unknowns, 1e15 times the others, meet zero
    columns in every coupling product.  Without refinement the others solve A x = b
    to the rounding of an FP32 elimination: |A x - b| <= h 2^-24 |A| |x| by column."""
    fosb, ctx, torch, m = fz
    n, h = m.n_edges, m.n_edges - 2048
    g = torch.Generator().manual_seed(5)
    A = torch.randn((h, h), dtype=torch.complex128, generator=g).to(ctx.torch_device)
    A = (A + A.T) / h ** 0.5 + 4.0 * torch.eye(h, dtype=A.dtype, device=A.device)
    Z = 1e-15 * torch.eye(n, dtype=A.dtype, device=A.device)
    Z[:h, :h] = A
    lv = fosb.Level(ctx, m, 1.0, Z, fosb.MIXED, opts=fosb.opts_default(lu_pivoting=pivoting, ir_max_sweeps=0))
    B = _rhs(torch, Z.device, n, 2)
    for adjoint in (False, True):
        x, b = _solve(lv, adjoint, B)[:h], B[:h]
        R = torch.matmul(A.mH.contiguous() if adjoint else A, x) - b
        worst = float((R.norm(dim=0) / (A.norm() * x.norm(dim=0))).max())
        print(f"[gpu] unused rows, pivoting {pivoting}, adjoint {adjoint}: residual {worst:.1e}", flush=True)
        assert worst <= h * 2.0 ** -24
    lv.close()


def test_trim_returns_packed_operands(fz):
    """The coupling of 3584 by 4096 packs at least 12 * 3584 * 4096 bytes, which a
    trim gives back; solves go on afterwards with the same result."""
    fosb, ctx, torch, m = fz
    Z = fosb.assemble(ctx, m, 2.0)
    lv = fosb.Level(ctx, m, 2.0, Z, fosb.MIXED)
    B = _rhs(torch, Z.device, m.n_edges, 4)
    X = _solve(lv, False, B)
    before = ctx.memory()["bytes_in_use"]
    ctx.trim()
    after = ctx.memory()
    assert after["bytes_in_use"] <= before - 12 * 3584 * 4096 and after["bytes_cached"] == 0
    assert torch.equal(X, _solve(lv, False, B))
    lv.close()


def _fill(torch, dev, leave):
    """Blocks that leave about that many bytes of the device free.  What is
    reported free can change by several hundred MB as blocks are taken, so this goes on
    until the report agrees."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    blocks = []
    for _ in range(64):
        room = torch.cuda.mem_get_info()[0] - leave
        if room < 4 << 20:
            break
        try:
            blocks.append(torch.empty(room, dtype=torch.uint8, device=dev))
        except torch.OutOfMemoryError:
            blocks.append(torch.empty(min(room, 64 << 20) // 2, dtype=torch.uint8, device=dev))
    free = torch.cuda.mem_get_info()[0]
    print(f"[gpu] {free / 2 ** 20:.0f} MiB free (asked for {leave / 2 ** 20:.0f})", flush=True)
    if abs(free - leave) >= 8 << 20:
        pytest.skip("the device could not be filled to the byte")
    return blocks


def test_calls_fit_without_the_optional_buffers(fz):
    """The packed operands and the 1024-row leaf inverses are not asked of a device
    that has no room for them: beside a block that leaves 230 MB (the level check
    asks for 200, its grown inverses and packed panels would take 230 beside the 35
    of the rest), then the work buffers of a wide solve (80 bytes an entry) and
    100 MB, less than the packed coupling's 188, level and solve succeed."""
    fosb, ctx, torch, m_ = fz
    dev, n = ctx.torch_device, m_.n_edges
    low = fosb.Context(0)
    fosb.autotune(low, 0)   # no scratch output for timing either
    m = fosb.Mesh(low, *workloads.geodesic_sphere(16))
    Z = fosb.assemble(low, m, 2.0)
    Zlow = torch.empty((n, n), dtype=torch.complex64, device=dev)
    fosb.Level(low, m, 2.0, Z, fosb.MIXED, Zlow=Zlow).close()   # the streams and kernels exist before the device fills up
    low.trim()
    ctx.trim()
    B = _rhs(torch, dev, n, 4)
    X = B.clone()
    ballast = _fill(torch, dev, 230 << 20)
    lv = fosb.Level(low, m, 2.0, Z, fosb.MIXED, Zlow=Zlow)
    del ballast
    low.trim()
    ballast = _fill(torch, dev, 80 * n * NRHS + (100 << 20))
    X.copy_(B)
    lv.solve(X)
    del ballast
    torch.cuda.empty_cache()
    R = torch.matmul(Z, X) - B
    assert float((R.norm(dim=0) / (Z.norm() * X.norm(dim=0))).max()) < 1e-9
    lv.close()
    low.close()


def test_workspace_query_covers_a_wide_solve(fz):
    """All that a fresh context's pools hold after a level and a solve with 2600
    columns (packed operands included) is within the query's bytes and the mesh's
    tables (under 16 MiB)."""
    fosb, ctx, torch, m_ = fz
    Z = fosb.assemble(ctx, m_, 2.0)
    own = fosb.Context(0)
    m = fosb.Mesh(own, *workloads.geodesic_sphere(16))
    lv = fosb.Level(own, m, 2.0, Z, fosb.MIXED)
    X = torch.randn((m.n_edges, 2600), dtype=torch.complex128, device=Z.device)
    lv.solve(X)
    mem = own.memory()
    level, work = fosb.level_workspace_size(m, fosb.MIXED, 1, 2600)
    held = mem["bytes_in_use"] + mem["bytes_cached"]
    print(f"[gpu] held {held / 2 ** 20:.0f} MiB, query {(level + work) / 2 ** 20:.0f} MiB", flush=True)
    assert held <= level + work + (16 << 20)
    lv.close()
    own.close()


def test_non_finite_entries_spread(fz):
    """A right-hand side column with an infinity or a NaN gives no finite column (or
    no convergence), and zero columns stay zero."""
    fosb, ctx, torch, m = fz
    Z = fosb.assemble(ctx, m, 2.0)
    lv = fosb.Level(ctx, m, 2.0, Z, fosb.MIXED, opts=fosb.opts_default(ir_max_sweeps=0))
    B = _rhs(torch, Z.device, m.n_edges, 3)
    B[7, 3], B[9, 5], B[:, 8] = float("inf"), float("nan"), 0.0
    X = _solve(lv, False, B)
    bad = ~torch.isfinite(torch.view_as_real(X)).all(dim=2).all(dim=0)
    assert bool(bad[3]) and bool(bad[5]) and int(bad.sum()) == 2
    assert float(X[:, 8].abs().max()) == 0.0
    lv.close()
