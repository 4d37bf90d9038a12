"""Tile kernels of the blocked LU at the sizes where they can go wrong: one
tile, tile and block edges, remainders, and the first size whose trailing
updates are split between the two streams.  A caller's matrix takes the pivoting
panels (tile inverses formed from the factored block), an assembled one the
speculative panels; both solve directions read the solve-ready form.

Matrices 2 I + G / sqrt(n) with G complex Gaussian of unit variance have a
2-norm condition number below 10, so the bound 8 n eps on the relative error of
the solution leaves the growth of rounding errors in an n-step elimination
(sqrt(n) in practice, n in the worst case) a factor of several.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2505_09545_amd import gdm
    c = gdm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 100, 127, 128, 129, 143, 256, 273, 700, 1900])
def test_getrf_getrs_tile_edges(ctx, n, dtype):
    rng = np.random.default_rng(n)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    A = A[rng.permutation(n)]  # the diagonal is no pivot
    B = rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))
    tol = 8 * max(n, 16) * (2.2e-16 if dtype == torch.complex128 else 1.2e-7)
    F = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype).contiguous()  # column-major storage
    ctx.getrf(F)
    for trans in (0, 1):
        X = torch.as_tensor(B).to(device="cuda", dtype=dtype).contiguous()
        ctx.getrs(F, X, trans)
        ref = np.linalg.solve(A.T if trans else A, B.T).T
        err = np.linalg.norm(X.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= tol, (n, dtype, trans, err)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(1, 1, 1), (5, 1, 1), (4, 4, 1), (43, 1, 1), (8, 8, 2), (43, 3, 1), (10, 10, 6), (9, 9, 8)])
def test_speculative_tile_edges(ctx, dims, prec):
    """n = 3 .. 1944 unknowns of dielectric boxes: the solution against LAPACK on
    the matrix that the library itself assembles (condition numbers below 100:
    1e-12 leaves 45 eps times that)."""
    import gdm_inputs as gi
    rng = np.random.default_rng(7)
    r = gi.cuboid_cells(*dims, 7.0)
    eps = rng.uniform(2.0, 9.0, len(r)) + 1j * rng.uniform(0.0, 0.5, len(r))
    k, e0 = gi.random_planewaves(rng, 3)
    before = ctx.pivot_fallbacks()
    ctx.set_environment(1.1)
    ctx.set_structure(r, 7.0, eps)
    M = ctx.assemble(640.0).cpu().numpy()
    ctx.factorize(640.0, prec)
    f0 = ctx.incident_planewave(k, e0)
    _, f = ctx.solve(f0)
    ref = np.linalg.solve(M, f0.cpu().numpy().T).T
    err = np.linalg.norm(f.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 1e-12, (dims, prec, err)
    assert ctx.pivot_fallbacks() == before


def test_getrf_fp32_column_scales(ctx):
    """Columns scaled by powers of two from 2^-80 to 1 (far outside the range of the
    16-bit operands of the FP32 updates): the pivots and every rounding stay the
    same, so D X of the scaled system (A D) X = B meets the same bound.  (Not for
    columns scaled up: the solve-ready form keeps I - U11^-1, which holds an entry
    of U11^-1 to 2^-24 only.)"""
    n = 700
    rng = np.random.default_rng(3)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    A = A[rng.permutation(n)]
    D = 2.0 ** rng.integers(-80, 1, n)
    B = rng.standard_normal((2, n)) + 1j * rng.standard_normal((2, n))
    F = torch.as_tensor((A * D[None, :]).T.copy()).to(device="cuda", dtype=torch.complex64).contiguous()
    X = torch.as_tensor(B).to(device="cuda", dtype=torch.complex64).contiguous()
    ctx.getrf(F)
    ctx.getrs(F, X, 0)
    ref = np.linalg.solve(A, B.T).T
    err = np.linalg.norm(X.cpu().numpy() * D[None, :] - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 8 * n * 1.2e-7, err


@pytest.mark.parametrize("dtype,n,nrhs", [(d, n, r) for d in (torch.complex64, torch.complex128)
                                          for n, r in ((5, 9), (16, 16), (64, 17), (65, 33), (127, 32), (129, 66), (300, 40),
                                                       (700, 9), (700, 131))])
def test_solve_step_edges(ctx, dtype, n, nrhs):
    """Block steps of the solves with more than eight right-hand sides at the edges
    of their 16-row and 32-column tiles, k of 64 and below; the bound of
    test_getrf_fp32_column_scales in each precision."""
    eps = 1.2e-7 if dtype == torch.complex64 else 2.3e-16
    rng = np.random.default_rng(n + nrhs)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    B = rng.standard_normal((nrhs, n)) + 1j * rng.standard_normal((nrhs, n))
    F = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype).contiguous()
    X = torch.as_tensor(B).to(device="cuda", dtype=dtype).contiguous()
    ctx.getrf(F)
    ctx.getrs(F, X, 0)
    ref = np.linalg.solve(A, B.T).T
    err = np.linalg.norm(X.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 8 * max(n, 16) * eps, err


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("n", [2, 16, 17, 33, 127, 150, 520, 2100])
def test_panel_pivots(ctx, n, dtype):
    """Pivots of the searching panels at the edges of their 16-column steps and
    workgroups (32 rows), against LAPACK's (the same |re| + |im|; Gaussian entries,
    whose largest differ by far more than the rounding here)."""
    from scipy.linalg import lu_factor
    rng = np.random.default_rng(7 * n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    F = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype).contiguous()
    piv = ctx.getrf(F).cpu().numpy()
    ref = lu_factor(A.astype(np.complex128 if dtype == torch.complex128 else np.complex64))[1]
    assert np.array_equal(piv, ref), np.nonzero(piv != ref)[0][:5]


def test_panels_of_many_and_few_rows(ctx):
    """n = 8300 in FP32: the first blocks have more rows per workgroup than a wave
    has lanes, the later ones fewer; the residual of one solve in FP64."""
    n = 8300
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn(n, n, dtype=torch.complex64, device="cuda", generator=g) / n ** 0.5
    A += 2 * torch.roll(torch.eye(n, dtype=torch.complex64, device="cuda"), 17, 0)
    B = torch.randn(1, n, dtype=torch.complex64, device="cuda", generator=g)
    F, X = A.clone(), B.clone()
    ctx.getrf(F)
    ctx.getrs(F, X, 0)
    x, b = X[0].to(torch.complex128), B[0].to(torch.complex128)
    res = torch.zeros_like(b)
    for k in range(0, n, 1000):  # storage row k is column k of the matrix
        res += (A[k:k + 1000].to(torch.complex128) * x[k:k + 1000, None]).sum(0)
    assert float((res - b).norm() / b.norm()) <= 8 * n * 1.2e-7


@pytest.mark.parametrize("cells", [1, 21, 22, 85, 86, 171, 343])
def test_row_norm_edges(ctx, cells):
    """The infinity norm in the backward error (64 rows and 256 columns per
    workgroup): an unrefined FP32 solution's error of about 1e-7, whose residual
    keeps six digits."""
    import gdm_inputs as gi
    rng = np.random.default_rng(cells)
    r = gi.cuboid_cells(7, 7, 7, 7.0)[:cells]
    ctx.set_environment(1.0)
    ctx.set_structure(r, 7.0, rng.uniform(2.0, 14.0, cells) + 0.1j)
    M = ctx.assemble(640.0).cpu().numpy()
    ctx.factorize(640.0, 1)
    f0 = rng.standard_normal((1, ctx.n)) + 1j * rng.standard_normal((1, ctx.n))
    _, f = ctx.solve(torch.as_tensor(f0), tol=1.0)
    x = f.cpu().numpy()[0]
    res = np.abs(f0[0] - M @ x).max()
    be = res / (np.abs(M).sum(1).max() * np.abs(x).max() + np.abs(f0).max())
    assert abs(ctx.info.backward_err - be) <= 1e-6 * be + 1e-15, (ctx.info.backward_err, be)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("n,nrhs", [(1, 1), (64, 2), (65, 4), (127, 1), (129, 5), (140, 8), (300, 9), (513, 1), (700, 20)])
def test_few_column_steps(ctx, n, nrhs, dtype):
    """Both solves with 1, 2, 4 and 8 columns at a time, remainders of them, and
    the edges of 64 rows, 4 columns and 128-wide blocks: the bound above."""
    rng = np.random.default_rng(n + nrhs)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    A = A[rng.permutation(n)]
    B = rng.standard_normal((nrhs, n)) + 1j * rng.standard_normal((nrhs, n))
    F = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype).contiguous()
    ctx.getrf(F)
    for trans in (0, 1):
        X = torch.as_tensor(B).to(device="cuda", dtype=dtype).contiguous()
        ctx.getrs(F, X, trans)
        ref = np.linalg.solve(A.T if trans else A, B.T).T
        err = np.linalg.norm(X.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= 8 * max(n, 16) * (2.2e-16 if dtype == torch.complex128 else 1.2e-7), (trans, err)


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("n,rows,cols", [(256, "two", 0), (700, "two", 0), (273, "spread", 0), (700, "spread", 0),
                                         (300, "steps", 0), (273, "spread", 20), (1900, "steps", 20)])
def test_getrf_fp32_row_scales(ctx, n, rows, cols, trans):
    """Rows (and columns) scaled by powers of two within and across the 128-wide
    blocks of the updates, whose products then pair small entries of L with large
    ones of U: groups of 2^0 and 2^-30, exponents sorted from 0 to -60, halved
    64 times a block.  The scales fall along the diagonal of 2 I + G / sqrt n, so
    the pivots stay on it (shuffled) and every rounding is that of the unscaled
    matrix: the bound above holds for the solution with the scales undone."""
    rng = np.random.default_rng(n)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    R = {"two": np.where(np.arange(n) < 100, 0, -30), "spread": -np.sort(rng.integers(0, 61, n)),
         "steps": -(np.arange(n) % 128) // 2 * (np.arange(n) < 128) - 64 * (np.arange(n) >= 128)}[rows]
    R, C = 2.0 ** R, 2.0 ** -rng.integers(0, cols + 1, n)
    B = rng.standard_normal((2, n)) + 1j * rng.standard_normal((2, n))
    p = rng.permutation(n)  # the matrix is (R A C)[p]
    F = torch.as_tensor((R[:, None] * A * C[None, :])[p].T.copy()).to(device="cuda", dtype=torch.complex64).contiguous()
    ctx.getrf(F)
    if trans:  # (C A^T R) y = C b with y in the order of p
        X = torch.as_tensor(B * C).to(device="cuda", dtype=torch.complex64).contiguous()
        ctx.getrs(F, X, 1)
        got = np.empty_like(B)
        got[:, p] = X.cpu().numpy()
        got, ref = got * R, np.linalg.solve(A.T, B.T).T
    else:
        X = torch.as_tensor((B * R)[:, p]).to(device="cuda", dtype=torch.complex64).contiguous()
        ctx.getrs(F, X, 0)
        got, ref = X.cpu().numpy() * C, np.linalg.solve(A, B.T).T
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 8 * n * 1.2e-7, err


@pytest.mark.parametrize("dtype,lda", [(torch.complex128, 18_000_000), (torch.complex64, 36_000_000)])
def test_getrf_long_columns(ctx, dtype, lda):
    """17 columns so far apart that a 16 x 16 tile spans more than 2^32 bytes, in the
    middle of larger ones: solution to the bound above, the rest of the storage
    untouched."""
    n = 17
    rng = np.random.default_rng(5)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    A = A[rng.permutation(n)]
    F = torch.full((n, lda), 7.0, dtype=dtype, device="cuda")
    F[:, :n] = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype)
    ctx.getrf(F)
    B = rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))
    for trans in (0, 1):
        X = torch.as_tensor(B).to(device="cuda", dtype=dtype).contiguous()
        ctx.getrs(F, X, trans)
        ref = np.linalg.solve(A.T if trans else A, B.T).T
        err = np.linalg.norm(X.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= 8 * n * (2.2e-16 if dtype == torch.complex128 else 1.2e-7), (trans, err)
    assert all(bool((F[j, n:] == 7).all()) for j in range(n))


@pytest.mark.parametrize("dtype,n,nrhs", [(torch.complex64, 120, 3), (torch.complex64, 200, 1), (torch.complex64, 2000, 230),
                                          (torch.complex128, 250, 1), (torch.complex128, 400, 4), (torch.complex128, 500, 6),
                                          (torch.complex128, 1000, 3), (torch.complex128, 1500, 140)])
def test_transposed_sweeps(ctx, dtype, n, nrhs):
    """Both sides of the choice between pushing and gathering transposed sweeps (few
    blocks, many columns): the bound above."""
    rng = np.random.default_rng(n + nrhs)
    A = 2 * np.eye(n) + (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(2 * n)
    A = A[rng.permutation(n)]
    B = rng.standard_normal((nrhs, n)) + 1j * rng.standard_normal((nrhs, n))
    F = torch.as_tensor(A.T.copy()).to(device="cuda", dtype=dtype).contiguous()
    X = torch.as_tensor(B).to(device="cuda", dtype=dtype).contiguous()
    ctx.getrf(F)
    ctx.getrs(F, X, 1)
    ref = np.linalg.solve(A.T, B.T).T
    err = np.linalg.norm(X.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 8 * n * (2.2e-16 if dtype == torch.complex128 else 1.2e-7), err


@pytest.mark.parametrize("dims,parts", [((7, 10, 10), 2), ((5, 4, 3), 3), ((5, 4, 7), 3)])
def test_transposed_sweeps_without_interchanges(ctx, dims, parts):
    """The adjoint's solves on speculative FP64 factors: gradients of 102 plane waves
    in one call (n = 2100: gathered) against the sum of parts of 51 (pushed), of 9 in
    one (n = 420: pushed) against threes (gathered), and n = 180, gathered either way.
    Condition numbers below 100 leave 1e-11 a factor of 400 over eps times that."""
    import gdm_inputs as gi
    rng = np.random.default_rng(11)
    r = gi.cuboid_cells(*dims, 7.0)
    ctx.set_environment(1.1)
    ctx.set_structure(r, 7.0, rng.uniform(2.0, 6.0, len(r)) + 0.2j)
    before = ctx.pivot_fallbacks()
    ctx.factorize(640.0, 0)
    assert ctx.pivot_fallbacks() == before
    nr = 102 if len(r) > 500 else 9
    k, e0 = gi.random_planewaves(rng, nr)
    gs = torch.as_tensor(rng.uniform(0.5, 1.5, (nr, 3)))
    f0 = ctx.incident_planewave(k, e0)
    q, f = ctx.solve(f0)
    whole = [t.cpu().numpy() for t in ctx.adjoint(k, e0, f0, q, f, gs)]
    sums = [0.0] * 3
    for p in np.array_split(np.arange(nr), parts):
        got = ctx.adjoint(k[p], e0[p], f0[p], q[p], f[p], gs[p])
        sums = [a + t.cpu().numpy() for a, t in zip(sums, got)]
    for a, b in zip(whole, sums):
        assert np.linalg.norm(a - b) <= 1e-11 * np.linalg.norm(b)
