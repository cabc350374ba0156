"""GPU parity of the observables beyond the plain rates, through the C ABI.

* phonon linewidth P^{el-ph}_{q nu} (Transport Methods, phonon BTE) against
  ``oracle.linewidth`` in both mesh-sum forms, bitwise repeatable;
* polar long-range coupling (Electron Properties, g = g^S + g^L): L(q, nu),
  the interpolated g and the rates against ``oracle.polar`` / ``coupling`` / ``rates``;
* group velocities (Velocity) and adaptive smearing (Dirac delta and
  Smearing) against ``oracle.velocity`` / ``rates``;
* the 3-phonon coupling V3 (Phonon Properties) against ``oracle.phonon3``;
* Philox streams, network initialisation, the training-set builder and the
  row gather against ``oracle.rng`` / ``oracle.mlp``;
* the finiteness scan (PHOEBE_E_NUMERIC) and a too-small workspace budget
  (PHOEBE_E_NOMEM).
"""

import numpy as np
import pytest

import synth
from gpu_common import rel_err, torch_cuda, workload_params
from helpers import group_sum_g2
from oracle import constants, coupling, linewidth, mlp, phonon3, polar, rates, rng, velocity

pytestmark = pytest.mark.gpu

P_BOUND = 1e-9       # linewidth and rates, FP64 (entries above 1e-10 of the maximum)
G2_BOUND = 1e-11     # degenerate-group |g|^2 relative to the pair's maximum
V_BOUND = 1e-10      # velocities relative to max |v|
V3_BOUND = 1e-11     # |V3| relative to max |V3|


@pytest.fixture(scope="module")
def lib():
    torch_cuda()
    from paper_2111_14999_amd import Library
    L = Library(0)
    yield L
    L.close()


def _params(s, mesh, width=0.8, sigma=0.05):
    t = rates.mesh_tables(s, mesh)
    mu = float(np.median(t["eps"]))
    par = dict(mu=mu, kT=constants.kT_of(300.0), sigma=sigma, win_lo=mu - width,
               win_hi=mu + width, omega_min=1e-4)
    return t, par


def _lw(lib, ds, mesh, par, nm):
    torch = torch_cuda()
    P = torch.full((int(np.prod(mesh)), nm), -1.0, dtype=torch.float64, device="cuda")
    n = lib.phonon_linewidth(ds, mesh, par, P)
    torch.cuda.synchronize()
    return n, P.cpu().numpy()


# ---------------------------------------------------------------------------
# phonon linewidth
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("case", ["toy", "nW5-3x4x5", "nW16-2x3x4", "nW20-3x3x4"])
@pytest.mark.parametrize("form", ["direct", "factored"])
def test_linewidth_matches_oracle(lib, case, form):
    """nW20: the factorised form's two column tiles per mode."""
    from paper_2111_14999_amd import DeviceSystem
    if case == "toy":
        s = synth.config_c1()
        p = workload_params()["toy"]
        mesh = tuple(p["mesh"])
        par = dict(mu=p["mu"], kT=p["kT"], sigma=p["sigma"], win_lo=p["win_lo"],
                   win_hi=p["win_hi"], omega_min=p["omega_min"])
        t = rates.mesh_tables(s, mesh)
    else:
        nW, mesh = {"nW5-3x4x5": (5, (3, 4, 5)), "nW16-2x3x4": (16, (2, 3, 4)),
                    "nW20-3x3x4": (20, (3, 3, 4))}[case]
        s = synth.small_system(81, n_wannier=nW, n_atoms=5 if nW == 16 else 2, r=1)
        s.h_r *= 0.3
        t, par = _params(s, mesh)
    print(f"[linewidth {case} {form}] mesh {mesh}", flush=True)
    ref = linewidth.phonon_linewidth(s, mesh, tables=t, **par)
    ds = DeviceSystem.from_host(s)
    try:
        lib.set_mesh_sum(form)
        n, P = _lw(lib, ds, mesh, par, s.n_modes)
        n2, P2 = _lw(lib, ds, mesh, par, s.n_modes)
    finally:
        lib.set_mesh_sum("auto")
    assert n == len(ref["k_idx"])
    assert np.array_equal(P, P2), "two calls differ"
    mx, med, ab = rel_err(P, ref["P"])
    print(f"  P rel err max {mx:.3e} median {med:.3e} (abs below floor {ab:.1e})", flush=True)
    assert np.max(ref["P"]) > 0
    assert mx < P_BOUND
    assert ab < 1e-10 * np.max(ref["P"])


def test_linewidth_gamma_by_product_and_errors(lib):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem, PhoebeError
    s = synth.small_system(82, n_wannier=4, n_atoms=2, r=1)
    s.h_r *= 0.3
    mesh = (3, 3, 4)
    t, par = _params(s, mesh)
    ds = DeviceSystem.from_host(s)
    N = int(np.prod(mesh))
    P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
    G = torch.zeros((N, s.n_wannier), dtype=torch.float64, device="cuda")
    n = lib.phonon_linewidth(ds, mesh, par, P, gamma_out=G)
    torch.cuda.synchronize()
    ref = rates.scattering_rates(s, mesh, tables=t, **par)
    mx, _, _ = rel_err(G.cpu().numpy()[:n], ref["gamma"])
    assert mx < P_BOUND
    for prec in ("fp32", "bf16x3"):
        with pytest.raises(PhoebeError) as e:
            lib.phonon_linewidth(ds, mesh, par, P, precision=prec)
        assert e.value.status == -4
    with pytest.raises(PhoebeError) as e:
        lib.phonon_linewidth(ds, mesh, par, P, q_mesh=(3, 3, 5))
    assert e.value.status == -4


# ---------------------------------------------------------------------------
# polar long-range coupling
# ---------------------------------------------------------------------------
def _polar_system(seed=91, nW=4, nat=2):
    s = synth.small_system(seed, n_wannier=nW, n_atoms=nat, r=1)
    s.h_r *= 0.3
    return synth.add_polar(s, seed, alpha=3.0, g_max=3)


def test_polar_factor_matches_oracle(lib):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    from oracle.bands import phonon_modes
    s = _polar_system()
    q = np.random.default_rng(3).uniform(-1, 1, size=(40, 3))
    w, z, _ = phonon_modes(q, s.rd, s.phi_r, s.mass)
    l = coupling.phonon_length(w, s.mass, 1e-4)
    ref = polar.polar_factor(q, z, l, s.born, s.eps_inf, s.ewald_alpha, s.g_max)
    ds = DeviceSystem.from_host(s)
    L = torch.zeros((40, s.n_modes), dtype=torch.complex128, device="cuda")
    lib.polar_factor(ds, torch.from_numpy(q).cuda(), L)
    torch.cuda.synchronize()
    got = L.cpu().numpy()
    # L carries the phase of each eigenvector: compare |L| (generic q, no degenerate modes)
    err = np.max(np.abs(np.abs(got) - np.abs(ref))) / np.max(np.abs(ref))
    print(f"[polar L] max ||L| - |L_ref|| / max |L| = {err:.2e}", flush=True)
    assert err < 1e-12


def test_polar_coupling_matches_oracle(lib):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = _polar_system(92)
    rng_ = np.random.default_rng(5)
    k = rng_.uniform(-1, 1, size=(3, 3))
    q = rng_.uniform(-1, 1, size=(20, 3))
    ref = coupling.coupling(k, q, s)
    ds = DeviceSystem.from_host(s)
    nk, nq, nW, nm = 3, 20, s.n_wannier, s.n_modes
    g = torch.empty((nk, nq, nm, nW, nW), dtype=torch.complex128, device="cuda")
    lib.interp_g(ds, torch.from_numpy(k).cuda(), torch.from_numpy(q).cuda(), g)
    torch.cuda.synchronize()
    g = g.cpu().numpy()
    worst = 0.0
    for i in range(nk):
        for j in range(nq):
            a = group_sum_g2(g[i, j], ref["eps_k"][i], ref["eps_kq"][i, j], ref["omega_q"][j])
            b = group_sum_g2(ref["g"][i, j], ref["eps_k"][i], ref["eps_kq"][i, j], ref["omega_q"][j])
            worst = max(worst, np.max(np.abs(a - b)) / np.max(b))
    print(f"[polar g] worst group |g|^2 err / pair max = {worst:.2e}", flush=True)
    assert worst < G2_BOUND


def test_polar_coupling_mesh_form(lib):
    """The polar term on the full-mesh form of the interpolation: against the list form
    on the same q points (same bands and modes, so g itself agrees) and, through the
    gauge-invariant group sums, against the oracle."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = _polar_system(94, nW=5, nat=2)
    mesh = (4, 3, 4)
    N = int(np.prod(mesh))
    i0, r = np.divmod(np.arange(N), mesh[1] * mesh[2])
    i1, i2 = np.divmod(r, mesh[2])
    q = np.stack([i0 / mesh[0], i1 / mesh[1], i2 / mesh[2]], axis=1)
    k = np.random.default_rng(6).uniform(-1, 1, size=(2, 3))
    ds = DeviceSystem.from_host(s)
    nW, nm = s.n_wannier, s.n_modes
    gm = torch.empty((2, N, nm, nW, nW), dtype=torch.complex128, device="cuda")
    gl = torch.empty_like(gm)
    kd = torch.from_numpy(k).cuda()
    lib.interp_g_mesh(ds, kd, mesh, gm)
    lib.interp_g(ds, kd, torch.from_numpy(q).cuda(), gl)
    torch.cuda.synchronize()
    gm, gl = gm.cpu().numpy(), gl.cpu().numpy()
    d = np.max(np.abs(gm - gl)) / np.max(np.abs(gl))
    ref = coupling.coupling(k, q, s)
    worst = 0.0
    for i in range(2):
        for j in range(N):
            a = group_sum_g2(gm[i, j], ref["eps_k"][i], ref["eps_kq"][i, j], ref["omega_q"][j])
            b = group_sum_g2(ref["g"][i, j], ref["eps_k"][i], ref["eps_kq"][i, j], ref["omega_q"][j])
            worst = max(worst, np.max(np.abs(a - b)) / np.max(b))
    print(f"[polar g mesh form] vs list form {d:.2e}, group |g|^2 vs oracle {worst:.2e}", flush=True)
    assert d < 1e-12
    assert worst < G2_BOUND


@pytest.mark.parametrize("form", ["direct", "factored"])
@pytest.mark.parametrize("nW,nat", [(5, 2), (20, 2), (16, 5)])
def test_polar_rates_match_oracle(lib, form, nW, nat):
    """nW 20: the factorised form's two column tiles per mode (the overlap over both);
    nW 16 with 15 modes: the two-wave, eight-tile form of the line kernel."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = _polar_system(93, nW=nW, nat=nat)
    mesh = (3, 4, 4)
    t, par = _params(s, mesh)
    ref = rates.scattering_rates(s, mesh, tables=t, **par)
    ds = DeviceSystem.from_host(s)
    N = int(np.prod(mesh))
    gam = torch.zeros((N, s.n_wannier), dtype=torch.float64, device="cuda")
    try:
        lib.set_mesh_sum(form)
        n = lib.scatter_rates(ds, mesh, par, gam)
        P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
        lib.phonon_linewidth(ds, mesh, par, P)
    finally:
        lib.set_mesh_sum("auto")
    torch.cuda.synchronize()
    assert n == len(ref["k_idx"])
    mx, med, _ = rel_err(gam.cpu().numpy()[:n], ref["gamma"])
    refP = linewidth.phonon_linewidth(s, mesh, tables=t, **par)["P"]
    mp, _, _ = rel_err(P.cpu().numpy(), refP)
    # the polar term matters here: the rates without it differ
    s0 = synth.small_system(93, n_wannier=nW, n_atoms=nat, r=1)
    s0.h_r *= 0.3
    plain = rates.scattering_rates(s0, mesh, tables=t, **par)["gamma"]
    diff, _, _ = rel_err(plain, ref["gamma"])
    print(f"[polar rates {form} nW {nW}] Gamma err {mx:.2e} (median {med:.2e}), P err {mp:.2e}; "
          f"without the polar term {diff:.2e}", flush=True)
    assert diff > 1e-3
    assert mx < P_BOUND and mp < P_BOUND


# ---------------------------------------------------------------------------
# velocities and adaptive smearing
# ---------------------------------------------------------------------------
def test_velocities_match_oracle(lib):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(61, n_wannier=6, n_atoms=2, r=2)
    k = np.random.default_rng(3).uniform(-1, 1, size=(50, 3))
    eps, v = velocity.group_velocities(k, s.rh, s.h_r)
    ds = DeviceSystem.from_host(s)
    V = torch.zeros((50, s.n_wannier, 3), dtype=torch.float64, device="cuda")
    E = torch.zeros((50, s.n_wannier), dtype=torch.float64, device="cuda")
    lib.velocities(ds, torch.from_numpy(k).cuda(), V, eps_out=E)
    torch.cuda.synchronize()
    err = np.max(np.abs(V.cpu().numpy() - v)) / np.max(np.abs(v))
    print(f"[velocity] max |v - v_ref| / max |v| = {err:.2e}", flush=True)
    assert err < V_BOUND
    assert np.max(np.abs(E.cpu().numpy() - eps)) < 1e-12 * np.max(np.abs(eps))


@pytest.mark.parametrize("nW", [1, 3, 16, 17, 32])
def test_velocities_band_tiles(lib, nW):
    """One and two 16-band passes, full and ragged, against the oracle."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(90 + nW, n_wannier=nW, n_atoms=1, r=1)
    k = np.random.default_rng(nW).uniform(-1, 1, size=(7, 3))
    _, v = velocity.group_velocities(k, s.rh, s.h_r)
    V = torch.zeros((7, nW, 3), dtype=torch.float64, device="cuda")
    lib.velocities(DeviceSystem.from_host(s, with_coupling=False), torch.from_numpy(k).cuda(), V)
    torch.cuda.synchronize()
    assert np.max(np.abs(V.cpu().numpy() - v)) < V_BOUND * np.max(np.abs(v))


def test_velocities_degenerate_pair(lib):
    """Two orbitals degenerate on the k_x = k_y plane: the 2x2 velocity block is
    diagonalised per direction (closed form, and the oracle)."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    R = synth.box_vectors(1)
    h = np.zeros((27, 2, 2), dtype=np.complex128)
    idx = {tuple(r): i for i, r in enumerate(R)}
    t = 0.7
    h[idx[(1, 0, 0)], 0, 0] = h[idx[(-1, 0, 0)], 0, 0] = t
    h[idx[(0, 1, 0)], 1, 1] = h[idx[(0, -1, 0)], 1, 1] = t
    rng_ = np.random.default_rng(0)
    a = (rng_.standard_normal((2, 2)) + 1j * rng_.standard_normal((2, 2)))
    W, _ = np.linalg.qr(a)
    h = np.conj(W.T)[None] @ h @ W[None]   # a Wannier rotation mixes the two orbitals
    s = synth.small_system(1, n_wannier=2, n_atoms=1, r=1)
    s.rh, s.h_r = R, np.ascontiguousarray(h)
    kap = 0.13
    k = np.array([[kap, kap, 0.3], [0.21, 0.21, -0.4]])
    eps, v = velocity.group_velocities(k, s.rh, s.h_r)
    ds = DeviceSystem.from_host(s)
    V = torch.zeros((2, 2, 3), dtype=torch.float64, device="cuda")
    lib.velocities(ds, torch.from_numpy(k).cuda(), V)
    torch.cuda.synchronize()
    got = V.cpu().numpy()
    vx = -2 * t * np.sin(2 * np.pi * kap)
    closed = np.array([sorted([vx, 0.0]), sorted([vx, 0.0]), [0.0, 0.0]]).T   # [band, alpha]
    assert np.max(np.abs(got[0] - closed)) < 1e-12
    assert np.max(np.abs(got - v)) < 1e-12


@pytest.mark.parametrize("form", ["direct", "factored"])
@pytest.mark.parametrize("nW,nat", [(5, 2), (20, 2), (16, 5)])
def test_adaptive_rates_and_linewidth_match_oracle(lib, form, nW, nat):
    """nW 16 with 15 modes: the factorised line kernel's two-wave, eight-tile form with
    per-transition widths; nW 20: two column tiles per mode."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(94, n_wannier=nW, n_atoms=nat, r=1)
    s.h_r *= 0.3
    mesh = (4, 3, 4)
    t, par = _params(s, mesh, sigma=0.02)
    ad = dict(sigma_min=0.02, prefactor=1.3)
    ref = rates.scattering_rates(s, mesh, tables=t, adaptive=ad, **par)
    refP = linewidth.phonon_linewidth(s, mesh, tables=t, adaptive=ad, **par)["P"]
    ds = DeviceSystem.from_host(s)
    par_g = dict(par, smearing="adaptive", adaptive_scale=1.3)
    N = int(np.prod(mesh))
    gam = torch.zeros((N, s.n_wannier), dtype=torch.float64, device="cuda")
    P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
    try:
        lib.set_mesh_sum(form)
        n = lib.scatter_rates(ds, mesh, par_g, gam)
        lib.phonon_linewidth(ds, mesh, par_g, P)
    finally:
        lib.set_mesh_sum("auto")
    torch.cuda.synchronize()
    assert n == len(ref["k_idx"])
    mx, med, _ = rel_err(gam.cpu().numpy()[:n], ref["gamma"])
    mp, _, _ = rel_err(P.cpu().numpy(), refP)
    fixed = rates.scattering_rates(s, mesh, tables=t, **par)["gamma"]
    diff, _, _ = rel_err(fixed, ref["gamma"])
    print(f"[adaptive {form} nW {nW}] Gamma err {mx:.2e} (median {med:.2e}), P err {mp:.2e}; "
          f"fixed width differs by {diff:.2e}", flush=True)
    assert diff > 1e-3
    assert mx < P_BOUND and mp < P_BOUND


@pytest.mark.parametrize("nW,nat", [(2, 1), (7, 2), (9, 3), (16, 4), (13, 5), (17, 5), (32, 2)])
def test_line_column_padding(lib, nW, nat):
    """Mode and band counts that leave padding in the columns of the factorised form, whose
    transforms are not written: rates, polar rates and linewidths against the direct sum."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    mesh = (6, 3, 5)
    N = int(np.prod(mesh))
    for pol in (False, True):
        s = synth.small_system(61 + nW, n_wannier=nW, n_atoms=nat, r=1)
        if pol:
            s = synth.add_polar(s, 61 + nW, alpha=3.0, g_max=2)
        t, par = _params(s, mesh, sigma=0.2)
        ds = DeviceSystem.from_host(s)
        out = {}
        try:
            for form in ("direct", "factored"):
                lib.set_mesh_sum(form)
                gam = torch.zeros((N, nW), dtype=torch.float64, device="cuda")
                P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
                lib.scatter_rates(ds, mesh, par, gam)
                lib.phonon_linewidth(ds, mesh, par, P)
                out[form] = gam.cpu().numpy(), P.cpu().numpy()
        finally:
            lib.set_mesh_sum("auto")
        assert np.max(out["direct"][0]) > 0
        for a, b in zip(out["factored"], out["direct"]):
            assert rel_err(a, b)[0] < 1e-10


@pytest.mark.parametrize("nW,nat,mesh,scale,smin", [
    (6, 2, (70, 2, 3), 1.0, 0.01),   # more points a line than a wave has lanes
    (16, 5, (18, 3, 2), 0.5, 1e-4),  # two waves; groups that close before they are full
    (16, 5, (5, 2, 2), 8.0, 0.5),    # every band live everywhere: full groups and a remainder
    (20, 4, (17, 2, 3), 1.0, 0.01),  # two tiles a mode, pairs of bands
    (3, 1, (1, 4, 3), 1.0, 0.01),
])
def test_adaptive_band_groups(lib, nW, nat, mesh, scale, smin):
    """Several final bands on one list of points against the direct sum, which takes them
    by themselves: rates and linewidths."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(97 + nW, n_wannier=nW, n_atoms=nat, r=1)
    s.h_r *= 0.3
    t, par = _params(s, mesh, sigma=smin)
    par = dict(par, smearing="adaptive", adaptive_scale=scale)
    ds = DeviceSystem.from_host(s)
    N = int(np.prod(mesh))
    out = {}
    try:
        for form in ("direct", "factored"):
            lib.set_mesh_sum(form)
            gam = torch.zeros((N, nW), dtype=torch.float64, device="cuda")
            P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
            lib.scatter_rates(ds, mesh, par, gam)
            lib.phonon_linewidth(ds, mesh, par, P)
            out[form] = gam.cpu().numpy(), P.cpu().numpy()
    finally:
        lib.set_mesh_sum("auto")
    assert np.max(out["direct"][0]) > 0
    for a, b in zip(out["factored"], out["direct"]):
        assert rel_err(a, b)[0] < 1e-10


# ---------------------------------------------------------------------------
# 3-phonon coupling
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("nat", [1, 2])
def test_v3_matches_oracle(lib, nat):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem3
    s = synth.small_system(5 + nat, n_wannier=1, n_atoms=nat, r=1)
    r, phi3 = synth.third_order_constants(5 + nat, nat)
    s.r1, s.r2, s.phi3 = r, r, phi3
    g = np.random.default_rng(nat)
    q = g.uniform(-1, 1, size=(3, 3))
    qp = g.uniform(-1, 1, size=(7, 3))
    ref = phonon3.interp_v3(q, qp, s)
    d3 = DeviceSystem3.from_host(s, r, phi3)
    nm = 3 * nat
    V = torch.zeros((3, 7, nm, nm, nm), dtype=torch.complex128, device="cuda")
    W3 = torch.zeros((3, 7, nm), dtype=torch.float64, device="cuda")
    lib.interp_v3(d3, torch.from_numpy(q).cuda(), torch.from_numpy(qp).cuda(), V, omega_qpp=W3)
    torch.cuda.synchronize()
    got = V.cpu().numpy()
    err = np.max(np.abs(np.abs(got) - np.abs(ref["v3"]))) / np.max(np.abs(ref["v3"]))
    werr = np.max(np.abs(W3.cpu().numpy() - ref["omega_qpp"])) / np.max(ref["omega_qpp"])
    print(f"[V3 nat={nat}] max ||V3| - ref| / max = {err:.2e}; omega'' err {werr:.1e}", flush=True)
    assert err < V3_BOUND
    assert werr < 1e-10


@pytest.mark.parametrize("nat", [3, 4, 5, 6, 7, 8, 9, 10])
def test_v3_rotation_tiles(lib, nat):
    """Every mode count of the rotation kernel (whole and split over nu) against the oracle."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem3
    s = synth.small_system(50 + nat, n_wannier=1, n_atoms=nat, r=1)
    r, phi3 = synth.third_order_constants(50 + nat, nat)
    keep = np.flatnonzero(np.abs(r).sum(axis=1) <= 1)[:3]  # (three vectors: the oracle's size)
    r = np.ascontiguousarray(r[keep])
    phi3 = np.ascontiguousarray(phi3[np.ix_(keep, keep)])
    s.r1, s.r2, s.phi3 = r, r, phi3
    g = np.random.default_rng(nat)
    q, qp = g.uniform(-1, 1, size=(2, 3)), g.uniform(-1, 1, size=(3, 3))
    ref = np.abs(phonon3.interp_v3(q, qp, s)["v3"])
    nm = 3 * nat
    V = torch.zeros((2, 3, nm, nm, nm), dtype=torch.complex128, device="cuda")
    lib.interp_v3(DeviceSystem3.from_host(s, r, phi3), torch.from_numpy(q).cuda(),
                  torch.from_numpy(qp).cuda(), V)
    torch.cuda.synchronize()
    assert np.max(np.abs(np.abs(V.cpu().numpy()) - ref)) < V3_BOUND * np.max(ref)


def test_v3_q_batches(lib):
    """Several q in one product and rotation against one q at a time, which a workspace
    without room for more takes."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem3, Library
    nat, nq, nqp = 5, 5, 2050
    s = synth.small_system(3, n_wannier=1, n_atoms=nat, r=1)
    r, phi3 = synth.third_order_constants(3, nat)
    g = np.random.default_rng(3)
    q = torch.from_numpy(g.uniform(-1, 1, size=(nq, 3))).cuda()
    qp = torch.from_numpy(g.uniform(-1, 1, size=(nqp, 3))).cuda()
    d3 = DeviceSystem3.from_host(s, r, phi3)
    nm = 3 * nat
    V, one = (torch.zeros((nq, nqp, nm, nm, nm), dtype=torch.complex128, device="cuda")
              for _ in range(2))
    x_bytes = nqp * nm**3 * 16
    small = Library(0, workspace_budget=4 * x_bytes)  # (E, D and z of the 10,250 q'' take one)
    try:
        lib.interp_v3(d3, q, qp, V)
        small.interp_v3(d3, q, qp, one)
    finally:
        small.close()
    torch.cuda.synchronize()
    assert float((V - one).abs().max()) < 1e-13 * float(V.abs().max())


def test_v3_q_groups(lib):
    """Two batches of q and a last group of q smaller than the others (17 q: groups of 5, 5, 5
    and 1, then 1) against calls of one q."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem3
    nat, nq, nqp = 5, 17, 3900
    nm = 3 * nat
    assert (1 << 30) // (16 * nqp * nm**3) == 5
    s = synth.small_system(4, n_wannier=1, n_atoms=nat, r=1)
    r, phi3 = synth.third_order_constants(4, nat)
    g = np.random.default_rng(4)
    q = torch.from_numpy(g.uniform(-1, 1, size=(nq, 3))).cuda()
    qp = torch.from_numpy(g.uniform(-1, 1, size=(nqp, 3))).cuda()
    d3 = DeviceSystem3.from_host(s, r, phi3)
    V = torch.zeros((nq, nqp, nm, nm, nm), dtype=torch.complex128, device="cuda")
    one = torch.zeros((1, nqp, nm, nm, nm), dtype=torch.complex128, device="cuda")
    lib.interp_v3(d3, q, qp, V)
    for i in range(nq):
        lib.interp_v3(d3, q[i:i + 1].contiguous(), qp, one)
        assert float((V[i] - one[0]).abs().max()) < 1e-13 * float(one.abs().max()), i


# ---------------------------------------------------------------------------
# Philox streams, initialisation, training set, gather
# ---------------------------------------------------------------------------
def test_philox_streams_bit_exact(lib):
    torch = torch_cuda()
    u = torch.zeros(100_003, dtype=torch.float64, device="cuda")
    lib.philox_uniform(1234, 77, u)
    r = torch.zeros(50_001, dtype=torch.int32, device="cuda")
    lib.philox_randint(99, 5, 64_000, r)
    torch.cuda.synchronize()
    assert np.array_equal(u.cpu().numpy(), rng.uniform(1234, 77, 100_003))
    assert np.array_equal(r.cpu().numpy().astype(np.int64), rng.randint(99, 5, 50_001, 64_000))


@pytest.mark.parametrize("precision", ["fp64", "bf16"])
def test_mlp_init_bit_exact(lib, precision):
    torch = torch_cuda()
    n_in, width, depth = 22, 32, 3
    n = lib.mlp_param_count(n_in, width, depth)
    dt = torch.float64 if precision == "fp64" else torch.float32
    th = torch.full((n,), 7.0, dtype=dt, device="cuda")
    lib.mlp_init(th, n_in, width, depth, seed=17, precision=precision)
    torch.cuda.synchronize()
    ref = mlp.init_params_philox(17, n_in, width, depth)
    got = th.cpu().numpy()
    if precision == "fp64":
        assert np.array_equal(got, ref)
    else:
        assert np.array_equal(got, ref.astype(np.float32))


def test_training_set_matches_oracle(lib):
    torch = torch_cuda()
    g = np.random.default_rng(4)
    ns, nq, nm = 5, 301, 6
    D = g.exponential(size=(ns, nq, nm)) * (g.uniform(size=(ns, nq, nm)) > 0.3)
    T = D * g.lognormal(size=D.shape)
    Tt, Dt = torch.from_numpy(T).cuda(), torch.from_numpy(D).cuda()
    for max_samples in (10 ** 9, 1500):
        cap = 20_000
        o_s = torch.zeros(cap, dtype=torch.int32, device="cuda")
        o_q = torch.zeros_like(o_s)
        o_v = torch.zeros_like(o_s)
        o_y = torch.zeros(cap, dtype=torch.float32, device="cuda")
        n, c = lib.training_set(Tt, Dt, ns, 0.05, 1e-3, max_samples, 11, o_s, o_q, o_v, o_y)
        torch.cuda.synchronize()
        st, q, nu, y, c_ref = mlp.training_set(T, D, 0.05, 1e-3, max_samples, 11)
        assert n == len(st)
        assert np.array_equal(o_s.cpu().numpy()[:n], st)
        assert np.array_equal(o_q.cpu().numpy()[:n], q)
        assert np.array_equal(o_v.cpu().numpy()[:n], nu)
        assert abs(c - c_ref) <= 1e-13 * abs(c_ref)
        assert np.max(np.abs(o_y.cpu().numpy()[:n] - y) / np.maximum(np.abs(y), 1.0)) < 1e-6


def test_gather_rows_bit_exact(lib):
    torch = torch_cuda()
    from paper_2111_14999_amd import PhoebeError
    X = torch.randn(1000, 37, device="cuda", dtype=torch.float32)
    idx = torch.from_numpy(np.random.default_rng(2).integers(0, 1000, 4096).astype(np.int32)).cuda()
    out = torch.zeros(4096, 37, device="cuda", dtype=torch.float32)
    lib.gather_rows(X, idx, out)
    torch.cuda.synchronize()
    assert torch.equal(out, X[idx.long()])
    bad = idx.clone()
    bad[7] = 1000
    with pytest.raises(PhoebeError) as e:
        lib.gather_rows(X, bad, out)
    assert e.value.status == -1


# ---------------------------------------------------------------------------
# validation: non-finite inputs and a too-small budget
# ---------------------------------------------------------------------------
def test_check_finite_and_nomem():
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem, Library, PhoebeError
    s = synth.small_system(83, n_wannier=4, n_atoms=2, r=1)
    mesh = (3, 3, 3)
    t, par = _params(s, mesh)
    L = Library(0)
    try:
        ds = DeviceSystem.from_host(s)
        gam = torch.zeros((27, 4), dtype=torch.float64, device="cuda")
        L.set_check_finite(True)
        L.scatter_rates(ds, mesh, par, gam)          # finite inputs pass
        ds.g_rr[3, 5, 1, 2, 0] = complex(float("nan"), 0.0)
        with pytest.raises(PhoebeError) as e:
            L.scatter_rates(ds, mesh, par, gam)
        assert e.value.status == -5
        ds.g_rr[3, 5, 1, 2, 0] = 0.0
        ds.h_r[0, 0, 0] = complex(float("inf"), 0.0)
        with pytest.raises(PhoebeError) as e:
            L.electron_bands(ds, torch.zeros((2, 3), dtype=torch.float64, device="cuda"),
                             torch.zeros((2, 4), dtype=torch.float64, device="cuda"))
        assert e.value.status == -5
    finally:
        L.close()
    small = Library(0, workspace_budget=1 << 16)
    try:
        ds = DeviceSystem.from_host(s)
        gam = torch.zeros((27, 4), dtype=torch.float64, device="cuda")
        with pytest.raises(PhoebeError) as e:
            small.scatter_rates(ds, mesh, par, gam)
        assert e.value.status == -2
        assert "budget" in str(e.value)
    finally:
        small.close()


@pytest.mark.parametrize("nat", [2, 3, 5])
def test_v3_modes_near_gamma(lib, nat):
    """V3 is that of the modes phonon_modes hands out, also where q'' comes so near Gamma that
    the rounding of D decides what its acoustic modes are: the contraction in numpy with
    the library's own modes."""
    torch = torch_cuda()
    from oracle.coupling import phonon_length
    from paper_2111_14999_amd import DeviceSystem, DeviceSystem3
    s = synth.small_system(50 + nat, n_wannier=1, n_atoms=nat, r=1)
    r, phi3 = synth.third_order_constants(50 + nat, nat)
    keep = np.flatnonzero(np.abs(r).sum(axis=1) <= 1)
    r = np.ascontiguousarray(r[keep])
    phi3 = np.ascontiguousarray(phi3[np.ix_(keep, keep)])
    g = np.random.default_rng(nat)
    q = g.uniform(-0.5, 0.5, size=(3, 3))
    qp = np.concatenate([-q + x * g.standard_normal((3, 3)) for x in (1e-3, 1e-4, 1e-5)])
    nm, omega_min = 3 * nat, 1e-9
    V = torch.zeros((3, 9, nm, nm, nm), dtype=torch.complex128, device="cuda")
    lib.interp_v3(DeviceSystem3.from_host(s, r, phi3), torch.from_numpy(q).cuda(),
                  torch.from_numpy(qp).cuda(), V, omega_min=omega_min)
    ds = DeviceSystem.from_host(s, with_coupling=False)

    def zl(pts):
        om = torch.zeros((len(pts), nm), dtype=torch.float64, device="cuda")
        z = torch.zeros((len(pts), nm, nm), dtype=torch.complex128, device="cuda")
        lib.phonon_modes(ds, torch.from_numpy(pts).cuda(), om, z)
        om, z = om.cpu().numpy(), z.cpu().numpy()
        return z * np.repeat(phonon_length(om, s.mass, omega_min), 3, axis=1)

    e1, e2 = zl(q), zl(qp)
    e3 = zl(-(q[:, None] + qp[None]).reshape(-1, 3)).reshape(3, 9, nm, nm)
    S = np.einsum("ir,rsabc->isabc", np.exp(-2j * np.pi * (q @ r.T)), phi3)
    X = np.einsum("js,isabc->ijabc", np.exp(-2j * np.pi * (qp @ r.T)), S)
    ref = np.einsum("ijabc,iau,jbv,ijcw->ijuvw", X, np.conj(e1), np.conj(e2), np.conj(e3), optimize=True)
    # pair by pair: the lengths of the lowest modes grow as q'' falls
    err = np.abs(V.cpu().numpy() - ref).max(axis=(2, 3, 4)) / np.abs(ref).max(axis=(2, 3, 4))
    assert err.max() < V3_BOUND


@pytest.mark.parametrize("nW,nat,mesh", [(3, 1, (7, 3, 4)), (4, 1, (20, 2, 3)), (6, 2, (18, 2, 3)), (20, 3, (6, 3, 2))])
@pytest.mark.parametrize("smearing", ["gaussian", "adaptive"])
def test_line_extensions_together(lib, nW, nat, mesh, smearing):
    """Polar terms with linewidths, adaptive widths and both, one atom (one band a list) and
    several, against the direct sum."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(97 + nW, n_wannier=nW, n_atoms=nat, r=1)
    s.h_r *= 0.3
    s = synth.add_polar(s, 97 + nW, alpha=3.0, g_max=2)
    t, par = _params(s, mesh, sigma=0.02)
    if smearing == "adaptive":
        par = dict(par, smearing="adaptive", adaptive_scale=1.0)
    ds = DeviceSystem.from_host(s)
    N = int(np.prod(mesh))
    out = {}
    try:
        for form in ("direct", "factored"):
            lib.set_mesh_sum(form)
            gam = torch.zeros((N, nW), dtype=torch.float64, device="cuda")
            P = torch.zeros((N, s.n_modes), dtype=torch.float64, device="cuda")
            lib.scatter_rates(ds, mesh, par, gam)
            lib.phonon_linewidth(ds, mesh, par, P)
            out[form] = gam.cpu().numpy(), P.cpu().numpy()
    finally:
        lib.set_mesh_sum("auto")
    assert np.max(out["direct"][0]) > 0
    for a, b in zip(out["factored"], out["direct"]):
        assert rel_err(a, b)[0] < 1e-10


@pytest.mark.parametrize("nW,nat,mesh", [(6, 2, (37, 3, 2)), (16, 4, (40, 2, 1)), (20, 3, (33, 2, 2))])
def test_adaptive_line_bytes(lib, nW, nat, mesh):
    """The bytes recorded for the line kernel with adaptive widths: T2 of every live line and the
    eigenvector rows of each list's bands at its units of 16 points, lists formed by the
    kernel's rule from the oracle's tables."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem, Library
    s = synth.small_system(140 + nW, n_wannier=nW, n_atoms=nat, r=1)
    s.h_r *= 0.3
    t, par = _params(s, mesh, sigma=0.002)
    par = dict(par, smearing="adaptive", adaptive_scale=0.4, win_lo=-1e30, win_hi=1e30)
    n0, n1, n2 = mesh
    N, NL = n0 * n1 * n2, n1 * n2
    idx = np.arange(N)
    pts = np.stack([idx // NL / n0, idx // n2 % n1 / n1, idx % n2 / n2], axis=1)
    v = velocity.group_velocities(pts, s.rh, s.h_r)[1]
    wmax = np.max(t["omega"])
    k_idx, most = np.array([0, 17, N - 1]), 2 if nW > 16 else 3
    lines = units = 0
    for k in k_idx:
        kk = np.array([k // NL, k // n2 % n1, k % n2])
        for n in range(nW):
            for q1 in range(n1):
                for q2 in range(n2):
                    kq = ((kk[0] + np.arange(n0)) % n0) * NL + (kk[1] + q1) % n1 * n2 + (kk[2] + q2) % n2
                    sg = velocity.adaptive_sigma(v[k, n], v[kq], mesh, 0.002, 0.4)  # [n0, nW]
                    live = np.abs(t["eps"][k, n] - t["eps"][kq]) <= 27.5 * sg + wmax
                    left = list(np.flatnonzero(live.any(axis=0)))
                    lines += len(left) > 0
                    of = lambda g: -(-int(live[:, g].any(axis=1).sum()) // 16)
                    while left:
                        g = [left.pop(0)]
                        while left and len(g) < most:
                            joined = of(g + [left[0]])
                            if joined * (3 + len(g)) > of(g) * (2 + len(g)) + 3 * of([left[0]]):
                                break
                            g.append(left.pop(0))
                        units += len(g) * of(g)
    own = Library(0)
    try:
        own.set_mesh_sum("factored")
        own.set_timing(True)
        gam = torch.zeros((3, nW), dtype=torch.float64, device="cuda")
        own.scatter_rates(DeviceSystem.from_host(s), mesh, par, gam,
                          k_idx=torch.from_numpy(k_idx.astype(np.int32)).cuda())
        got = own.kernel_bytes("line_rates")
    finally:
        own.close()
    assert got == 16.0 * 3 * s.n_modes * nW * lines + 16.0 * nW * 16 * units
