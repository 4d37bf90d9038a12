"""The dyad as the per-pair kernels evaluate it (reciprocal square root, two-part
phase, own sine and cosine): probe fields from a fraction of the step to kR of
about 10^5, in a medium, for cells and effective dipoles; and the far-field
double sum at its tile, split and right-hand-side remainders."""
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


@pytest.mark.parametrize("dist", [0.6, 9.0, 250.0, 4.1e4, 7.3e6])
def test_fields_over_distance(ctx, dist):
    """Bound: the oracle and the kernel each round the phase kR (relative 2^-53 of
    it, a few roundings) and a handful of products: 16 eps (10 + kR)."""
    import gdm_inputs as gi
    from oracle import gdm_oracle as O
    w = gi.small_mixed()
    n_env, wl = w["n_env"], w["wavelength"]
    rng = np.random.default_rng(1)
    v = rng.standard_normal((40, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    pos = np.concatenate([w["r_cell"], w["r_eff"]])
    probes = pos[rng.integers(len(pos), size=40)] + dist * v
    ctx.set_environment(n_env)
    ctx.set_structure(w["r_cell"], w["step"], w["eps_cell"], w["r_eff"], w["alpha_eff"])
    ctx.set_wavelength(wl)
    q = rng.standard_normal((3, ctx.n)) + 1j * rng.standard_normal((3, ctx.n))
    E, H = ctx.fields(torch.as_tensor(q), torch.as_tensor(probes))
    D = O.Dipoles(w)
    Es, Hs = O.scattered_fields(D, q.T, probes)
    tol = 16 * 2.2e-16 * (10 + 2 * np.pi / wl * n_env * (dist + 400.0))
    for got, ref in ((E.cpu().numpy(), Es), (H.cpu().numpy(), Hs)):
        err = np.linalg.norm(got - ref, axis=(1, 2)) / np.linalg.norm(ref, axis=(1, 2))
        assert err.max() <= tol, (dist, err, tol)


@pytest.mark.parametrize("cells,eff,nrhs", [(1, 0, 1), (1, 0, 2), (63, 2, 5), (64, 0, 4), (65, 1, 1), (257, 0, 3), (260, 70, 9)])
def test_far_field_sum_edges(ctx, cells, eff, nrhs):
    """Random moments; the double sum adds N^2 terms in another order than the
    oracle: 1e-12 of the sum of their moduli is over 100 times the rounding."""
    import gdm_inputs as gi
    from oracle import gdm_oracle as O
    rng = np.random.default_rng(cells + eff)
    r = gi.cuboid_cells(7, 7, (cells + 48) // 49, 6.0)[:cells]
    re = np.stack([150.0 + 90.0 * np.arange(eff), np.zeros(eff), 30.0 * (np.arange(eff) % 3)], 1)
    k, e0 = gi.random_planewaves(rng, nrhs)
    w = dict(r_cell=r, step=6.0, eps_cell=np.full(cells, 5.0 + 0.2j), n_env=1.2, wavelength=600.0, r_eff=re,
             alpha_eff=gi.mie_like_alpha6(rng, eff, 600.0, 1.2), khat=k, e0=e0, r_probe=np.zeros((0, 3)))
    ctx.set_environment(1.2)
    ctx.set_structure(r, 6.0, w["eps_cell"], re if eff else None, w["alpha_eff"] if eff else None)
    ctx.set_wavelength(600.0)
    q = rng.standard_normal((nrhs, ctx.n)) + 1j * rng.standard_normal((nrhs, ctx.n))
    t = torch.as_tensor(q)
    cs = ctx.cross_sections(t, t, t, torch.ones(nrhs, dtype=torch.float64), want_ff=True).cpu().numpy()
    D = O.Dipoles(w)
    ref = O.sca_farfield_doublesum(D, q.T, np.ones(nrhs))
    scale = np.abs(O.cross_sections(D, q.T, q.T, q.T, np.ones(nrhs))["rad"]) + np.abs(ref)
    # near-field terms cancel in the imaginary part: their size relative to the radiated power is below 1e4 here
    assert np.max(np.abs(cs[:, 4] - ref) / scale) <= 1e-9, (cs[:, 4], ref)


@pytest.mark.parametrize("cells,eff,nrhs", [(63, 2, 5), (65, 1, 1), (257, 0, 3), (260, 70, 9)])
def test_far_field_sum_against_its_terms(ctx, cells, eff, nrhs):
    """The same sum against the size of its own terms.  Both sides round a dyad to
    eps (10 + kR) of its norm (kR below 100 here) and add N terms per target one
    after another: 2.2e-16 (110 + 330) < 1e-13 of sum_ij |q_i| |G_ij| |q_j| on each
    side; 1e-12 leaves a factor of five over both."""
    import gdm_inputs as gi
    from oracle import gdm_oracle as O
    rng = np.random.default_rng(cells + eff)
    r = gi.cuboid_cells(7, 7, (cells + 48) // 49, 6.0)[:cells]
    re = np.stack([150.0 + 90.0 * np.arange(eff), np.zeros(eff), 30.0 * (np.arange(eff) % 3)], 1)
    k, e0 = gi.random_planewaves(rng, nrhs)
    w = dict(r_cell=r, step=6.0, eps_cell=np.full(cells, 5.0 + 0.2j), n_env=1.2, wavelength=600.0, r_eff=re,
             alpha_eff=gi.mie_like_alpha6(rng, eff, 600.0, 1.2), khat=k, e0=e0, r_probe=np.zeros((0, 3)))
    ctx.set_environment(1.2)
    ctx.set_structure(r, 6.0, w["eps_cell"], re if eff else None, w["alpha_eff"] if eff else None)
    ctx.set_wavelength(600.0)
    q = rng.standard_normal((nrhs, ctx.n)) + 1j * rng.standard_normal((nrhs, ctx.n))
    t = torch.as_tensor(q)
    cs = ctx.cross_sections(t, t, t, torch.ones(nrhs, dtype=torch.float64), want_ff=True).cpu().numpy()
    D = O.Dipoles(w)
    ref = O.sca_farfield_doublesum(D, q.T, np.ones(nrhs))
    R = D.pos[:, None, :] - D.pos[None, :, :]
    same = np.all(R == 0.0, axis=-1)
    g = np.linalg.norm(O.green6(np.where(same[..., None], 1.0, R), D.k0, D.n_env), axis=(2, 3))
    g[same] = 0.0
    size = np.linalg.norm(D.to6(q.T), axis=1)  # [N, rhs]
    terms = 4 * np.pi * D.k0 / D.n_env * np.einsum("ir,ij,jr->r", size, g, size)
    assert np.max(np.abs(cs[:, 4] - ref) / terms) <= 1e-12, (cs[:, 4], ref, terms)
