"""Error paths of the C-ABI forced from the host, every kernel exiting normally:
GDM_E_NOCONV from a refinement budget too small for the tolerance (single
system and batched spectra), GDM_E_OOM from a device-memory limit on the
context, and the binding's retry in halves after GDM_E_OOM (probe fields and
right-hand sides), whose results must equal those of an unlimited context.
"""
import sys

import numpy as np
import pytest

import gdm_inputs as gi
from oracle import gdm_oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def relcol(a, b):
    a = np.asarray(a).reshape(len(a), -1)
    b = np.asarray(b).reshape(len(b), -1)
    return float(np.max(np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)))


@pytest.fixture(scope="module")
def gdm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_09545_amd import gdm as g
    return g


def small_structure(n_rhs=2):
    """config-4 recipe at 4 x 5 x 6 cells (n = 360), plane waves along +z and
    tilted, 64 x 64 probes (four dipole splits of the probe sum)."""
    w = dict(gi.config4())
    w["r_cell"] = gi.cuboid_cells(4, 5, 6, 8.0)
    w["eps_cell"] = np.full(len(w["r_cell"]), 10.0 + 0.05j)
    k, e = gi.random_planewaves(np.random.default_rng(9), n_rhs)
    w["khat"], w["e0"] = k, e
    return w


def setup(ctx, w, prec):
    ctx.set_environment(w["n_env"])
    ctx.set_structure(torch.as_tensor(w["r_cell"]), w["step"], torch.as_tensor(w["eps_cell"]))
    ctx.factorize(w["wavelength"], prec)
    from paper_2505_09545_amd import gdm as g
    khat, e0, e2 = g.plane_wave_inputs(w, ctx)
    return ctx.incident_planewave(khat, e0)


def test_refinement_budget_too_small_reports_noconv(gdm):
    """FP32 factors with no FP64 correction allowed: the backward error of the
    FP32 solve (~1e-7) is above tol = 1e-14, so GDM_E_NOCONV, with the FP32
    iterate written (within FP32 accuracy of the oracle) and its backward error
    reported; one correction later the call succeeds."""
    w = small_structure()
    sim = O.simulate(w)
    ctx = gdm.Context(0)
    try:
        f0 = setup(ctx, w, gdm.PREC_FP32_IR)
        say("noconv: max_iter 0")
        with pytest.raises(gdm.GDMError) as ei:
            ctx.solve(f0, tol=1e-14, max_iter=0)
        assert ei.value.status == gdm.GDM_E_NOCONV
        assert ctx.info.ir_iters == 0 and 1e-14 < ctx.info.backward_err < 1e-5
        # the best iterate is still written: call the C entry point directly for the outputs
        import ctypes
        q = torch.full_like(f0, complex("nan"))
        st = ctx._call("gdm_solve", ctx.h, f0.shape[0], gdm._ptr(f0), 1e-14, 0, gdm._ptr(q), None,
                       ctypes.byref(ctx.info))
        assert st == gdm.GDM_E_NOCONV
        torch.cuda.synchronize()
        assert relcol(q.cpu().numpy(), sim["q"].T) < 1e-5
        q2, _ = ctx.solve(f0, tol=1e-14, max_iter=10)
        assert relcol(q2.cpu().numpy(), sim["q"].T) < 1e-10
    finally:
        ctx.close()


def test_memory_limit_reports_oom_and_lifts(gdm):
    w = small_structure()
    ctx = gdm.Context(0)
    try:
        with pytest.raises(gdm.GDMError) as ei:
            ctx.set_memory_limit(-1)
        assert ei.value.status == gdm.GDM_E_ARG
        ctx.set_environment(w["n_env"])
        ctx.set_structure(torch.as_tensor(w["r_cell"]), w["step"], torch.as_tensor(w["eps_cell"]))
        used = ctx.memory_used()
        # the 360 x 360 complex128 matrix alone is 2 MB
        ctx.set_memory_limit(used + (1 << 20))
        say("oom: factorize under a 1 MiB headroom")
        with pytest.raises(gdm.GDMError) as ei:
            ctx.factorize(w["wavelength"], gdm.PREC_FP64)
        assert ei.value.status == gdm.GDM_E_OOM
        assert ctx.memory_used() <= used + (1 << 20)
        ctx.set_memory_limit(0)
        ctx.factorize(w["wavelength"], gdm.PREC_FP64)
    finally:
        ctx.close()


def test_binding_retries_probe_halves_after_oom(gdm):
    """The probe sum's partial sums need 2 x 4 splits x 2 RHS x P x 48 B; with
    room for a quarter of the 4096 probes only, the binding evaluates them in
    quarters (two levels of halving), and the fields equal those of an
    unlimited context bit for bit (same kernels, same dipole splits)."""
    w = small_structure()
    rp = torch.as_tensor(gi.probe_plane(64, 64, 200.0, 200.0, -150.0), dtype=torch.float64)
    ref = gdm.Context(0)
    lim = gdm.Context(0)
    try:
        f0 = setup(ref, w, gdm.PREC_FP64)
        q, _ = ref.solve(f0)
        E_ref, H_ref = ref.fields(q, rp)
        setup(lim, w, gdm.PREC_FP64)
        need_full = 2 * 4 * q.shape[0] * len(rp) * 48
        lim.set_memory_limit(lim.memory_used() + need_full // 4 + 4096)
        say("oom retry: probes", len(rp), "headroom", need_full // 4 + 4096)
        E, H = lim.fields(q, rp)
        torch.cuda.synchronize()
        assert torch.equal(E, E_ref) and torch.equal(H, H_ref)
    finally:
        ref.close()
        lim.close()
    # when even one probe does not fit, the error reaches the caller
    one = gdm.Context(0)
    try:
        setup(one, w, gdm.PREC_FP64)
        one.set_memory_limit(one.memory_used() + 1)
        with pytest.raises(gdm.GDMError) as ei:
            one.fields(q, rp[:3])
        assert ei.value.status == gdm.GDM_E_OOM
    finally:
        one.close()


def test_binding_retries_rhs_halves_after_oom(gdm):
    """16 right-hand sides with room for the solve workspaces of 4 at a time:
    the binding solves them in quarters; moments within 1e-12 of an unlimited
    context (FP64 factors; the quarters take the few-RHS kernels)."""
    w = small_structure(n_rhs=16)
    ref = gdm.Context(0)
    lim = gdm.Context(0)
    try:
        f0 = setup(ref, w, gdm.PREC_FP64)
        q_ref, _ = ref.solve(f0)
        f0l = setup(lim, w, gdm.PREC_FP64)
        lim.solve(f0l[:1])  # allocates the one-RHS workspaces
        n = lim.n
        lim.set_memory_limit(lim.memory_used() + 4 * n * 16 + 1024)
        say("oom retry: 16 RHS, headroom for 4")
        q, _ = lim.solve(f0l)
        torch.cuda.synchronize()
        assert relcol(q.cpu().numpy(), q_ref.cpu().numpy()) < 1e-12
    finally:
        ref.close()
        lim.close()


def test_batch_noconv_when_corrections_fall_short(gdm):
    """Batched spectra with tol: no FP64 correction (ir_iters 0) leaves the
    FP32 backward error, GDM_E_NOCONV with every output written; two
    corrections reach 1e-13 and the call succeeds."""
    from test_gpu_batch import small_batch
    structs, wl, eps, khat, e0 = small_batch(n_wl=3)
    ctx = gdm.Context(0)
    try:
        ctx.set_environment(1.0)
        say("batch noconv: ir_iters 0")
        with pytest.raises(gdm.GDMError) as ei:
            ctx.batch_spectra(structs, 10.0, wl, eps, khat, e0, ir_iters=0, tol=1e-14)
        assert ei.value.status == gdm.GDM_E_NOCONV
        assert ctx.info.backward_err > 1e-14
        cs, be = ctx.batch_spectra(structs, 10.0, wl, eps, khat, e0, ir_iters=2, tol=1e-13)
        assert float(be.max()) <= 1e-13
        with pytest.raises(gdm.GDMError) as ei:
            ctx.batch_spectra(structs, 10.0, wl, eps, khat, e0, tol=-1.0)
        assert ei.value.status == gdm.GDM_E_ARG
    finally:
        ctx.close()


def test_buffers_of_one_call_yield_to_a_limit(gdm):
    """The split operands of an FP32 factorisation, the wide form of the iterative
    solver's workspace and the far-field sum's parts are given back, or done
    without, where a limit leaves no room: one byte less than an unlimited context
    holds after each call still serves it, refined results to the same tolerance
    (backward error 1e-14; condition numbers below 100: 1e-11)."""
    w = small_structure()
    n = 3 * len(w["r_cell"])

    def stages(ctx, limit):
        out = []
        ctx.set_environment(w["n_env"])
        ctx.set_structure(torch.as_tensor(w["r_cell"]), w["step"], torch.as_tensor(w["eps_cell"]))
        say("limit: factorize", limit[0])
        ctx.set_memory_limit(limit[0])
        ctx.factorize(w["wavelength"], gdm.PREC_FP32_IR)
        used = [ctx.memory_used()]
        khat, e0, e2 = gdm.plane_wave_inputs(w, ctx)
        f0 = ctx.incident_planewave(khat, e0)
        say("limit: solve", limit[1])
        ctx.set_memory_limit(limit[1])
        q, f = ctx.solve(f0)
        used.append(ctx.memory_used())
        out += [q, f]
        say("limit: far field", limit[2])
        ctx.set_memory_limit(limit[2])
        out.append(ctx.cross_sections(f0, q, f, e2, want_ff=True))
        used.append(ctx.memory_used())
        say("limit: iterative", limit[3])
        ctx.set_memory_limit(limit[3])
        out.append(ctx.solve_iterative(w["wavelength"], f0, restart=200)[0])
        used.append(ctx.memory_used())
        torch.cuda.synchronize()
        return used, [o.cpu().numpy() for o in out]

    ref, lim = gdm.Context(0), gdm.Context(0)
    try:
        used, a = stages(ref, [0] * 4)
        tight, b = stages(lim, [u - 1 for u in used])
    finally:
        ref.close()
        lim.close()
    assert all(t < u for t, u in zip(tight, used)), (tight, used)
    # the matrices, and no more than three buffers of n x 128 beside them
    assert tight[0] < 24 * n * n + 3 * max(n, 512) * 128 * 8 + (2 << 20)
    for x, y in zip(a, b):
        assert relcol(y, x) <= 1e-11


def test_batch_without_room_for_split_operands(gdm):
    """The same for batched spectra: 16 systems of n = 150, whose split operands
    take more than their matrices."""
    structs = [gi.cuboid_cells(5, 5, 2, 10.0)]
    wl = np.linspace(450.0, 800.0, 16)
    eps = (2.2 + 0.05j * np.arange(16))[None, :]
    khat, e0 = gi.normal_incidence_xy()
    ref, lim = gdm.Context(0), gdm.Context(0)
    try:
        for c in (ref, lim):
            c.set_environment(1.0)
        a, _ = ref.batch_spectra(structs, 10.0, wl, eps, khat, e0, prec=1)
        say("batch: limit one byte below", ref.memory_used())
        lim.set_memory_limit(ref.memory_used() - 1)
        b, be = lim.batch_spectra(structs, 10.0, wl, eps, khat, e0, prec=1)
        assert bool((be <= 1e-14).all())
        a, b = a.cpu().numpy(), b.cpu().numpy()
        assert np.max(np.abs(a - b) / a[..., :1]) <= 1e-11
    finally:
        ref.close()
        lim.close()
