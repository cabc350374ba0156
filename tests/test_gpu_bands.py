"""GPU band structure (phase tables + MFMA Fourier sum + batched Jacobi) vs the oracle.

Eigenvalues are compared with LAPACK's; eigenvectors through residuals
against the oracle's own H(k) and D(q) (any phase per vector is valid).
"""

import numpy as np
import pytest

import synth
from gpu_common import torch_cuda
from oracle import bands

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    torch_cuda()
    from paper_2111_14999_amd import Library
    L = Library(0)
    yield L
    L.close()


@pytest.mark.parametrize("make", [lambda: synth.config_c1(),
                                  lambda: synth.small_system(41, n_wannier=7, n_atoms=5, r=1),
                                  lambda: synth.small_system(42, n_wannier=1, n_atoms=1, r=2),
                                  lambda: synth.config_c2(with_coupling=False)],
                         ids=["toy", "nW7-5atoms", "nW1-1atom", "nW16-15modes"])
def test_electron_and_phonon_bands(lib, make):
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = make()
    ds = DeviceSystem.from_host(s, with_coupling=False)
    rng = np.random.default_rng(0)
    k = rng.uniform(-1, 1, size=(333, 3))
    k[0] = 0.0
    kd = torch.from_numpy(k).cuda()
    nW, nm = s.n_wannier, s.n_modes
    eps = torch.empty((k.shape[0], nW), dtype=torch.float64, device="cuda")
    U = torch.empty((k.shape[0], nW, nW), dtype=torch.complex128, device="cuda")
    lib.electron_bands(ds, kd, eps, U)
    w = torch.empty((k.shape[0], nm), dtype=torch.float64, device="cuda")
    z = torch.empty((k.shape[0], nm, nm), dtype=torch.complex128, device="cuda")
    lib.phonon_modes(ds, kd, w, z)
    torch.cuda.synchronize()
    eps, U, w, z = eps.cpu().numpy(), U.cpu().numpy(), w.cpu().numpy(), z.cpu().numpy()

    e_ref, _ = bands.electron_bands(k, s.rh, s.h_r)
    H = bands.hamiltonian_k(k, s.rh, s.h_r)
    scale = np.max(np.abs(e_ref))
    assert np.max(np.abs(eps - e_ref)) < 1e-12 * scale
    assert np.max(np.abs(H @ U - U * eps[:, None, :])) < 1e-12 * scale
    assert np.max(np.abs(np.conj(np.swapaxes(U, 1, 2)) @ U - np.eye(nW))) < 1e-12

    w_ref, _, lam = bands.phonon_modes(k, s.rd, s.phi_r, s.mass)
    D = bands.dynamical_matrix(k, s.rd, s.phi_r, s.mass)
    # hbar omega = C sqrt(lambda) amplifies rounding of lambda ~ 0 (acoustic at q = 0)
    big = w_ref > 1e-4
    assert np.max(np.abs(w[big] - w_ref[big]) / w_ref[big]) < 1e-10
    assert np.max(np.abs(w[~big] - w_ref[~big]), initial=0.0) < 1e-6
    res = D @ z - z * np.maximum(lam, 0)[:, None, :]
    assert np.max(np.abs(res)) < 1e-11 * np.max(np.abs(lam))
    assert np.max(np.abs(np.conj(np.swapaxes(z, 1, 2)) @ z - np.eye(nm))) < 1e-12


def test_degenerate_spectrum(lib):
    """H(R) = 0 except H(0) = diag with repeated values: exact degeneracies."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(43, n_wannier=6, n_atoms=1, r=1)
    s.h_r[:] = 0
    s.h_r[13] = np.diag([0.5, -1.0, 0.5, 2.0, -1.0, 0.5])
    ds = DeviceSystem.from_host(s, with_coupling=False)
    k = np.random.default_rng(1).uniform(-1, 1, size=(17, 3))
    kd = torch.from_numpy(k).cuda()
    eps = torch.empty((17, 6), dtype=torch.float64, device="cuda")
    lib.electron_bands(ds, kd, eps, None)
    torch.cuda.synchronize()
    ref = np.sort([0.5, -1.0, 0.5, 2.0, -1.0, 0.5])
    assert np.max(np.abs(eps.cpu().numpy() - ref[None])) < 1e-15


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 10, 11, 13, 16, 17, 19, 22, 23, 27, 31, 32])
def test_eigensolver_orders(lib, n):
    """Every layout of the eigensolver: matrices per wave (64 at order 1 down to one), waves per
    matrix, odd orders, a ragged last work-group, and equal diagonal entries (the sign of
    the first rotations)."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(70, n_wannier=n, n_atoms=1, r=1)
    s.h_r[13] -= np.diag(np.diag(s.h_r[13])) - 0.25 * np.eye(n)
    ds = DeviceSystem.from_host(s, with_coupling=False)
    k = np.random.default_rng(n).uniform(-1, 1, size=(67, 3))
    eps = torch.empty((67, n), dtype=torch.float64, device="cuda")
    U = torch.empty((67, n, n), dtype=torch.complex128, device="cuda")
    lib.electron_bands(ds, torch.from_numpy(k).cuda(), eps, U)
    torch.cuda.synchronize()
    eps, U = eps.cpu().numpy(), U.cpu().numpy()
    H = bands.hamiltonian_k(k, s.rh, s.h_r)
    ref = np.linalg.eigvalsh(H)
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(eps - ref)) < 1e-13 * scale
    assert np.max(np.abs(H @ U - U * eps[:, None, :])) < 1e-13 * scale
    assert np.max(np.abs(np.conj(np.swapaxes(U, 1, 2)) @ U - np.eye(n))) < 1e-13


@pytest.mark.parametrize("nat", [1, 2, 3, 4, 5, 6, 8, 10])
def test_phonon_solvers(lib, nat):
    """The solver of modes handed out, every order it has, against D(q) itself; frequencies
    alone go by the other one and agree."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(80 + nat, n_wannier=1, n_atoms=nat, r=1)
    ds = DeviceSystem.from_host(s, with_coupling=False)
    q = np.random.default_rng(nat).uniform(-1, 1, size=(67, 3))
    nm = 3 * nat
    om, only = (torch.empty((67, nm), dtype=torch.float64, device="cuda") for _ in range(2))
    z = torch.empty((67, nm, nm), dtype=torch.complex128, device="cuda")
    lib.phonon_modes(ds, torch.from_numpy(q).cuda(), om, z)
    lib.phonon_modes(ds, torch.from_numpy(q).cuda(), only)
    torch.cuda.synchronize()
    om, only, z = om.cpu().numpy(), only.cpu().numpy(), z.cpu().numpy()
    D = bands.dynamical_matrix(q, s.rd, s.phi_r, s.mass)
    lam = np.linalg.eigvalsh(D)
    scale = np.max(np.abs(lam))
    got = np.einsum("qin,qij,qjn->qn", np.conj(z), D, z).real
    assert np.max(np.abs(got - lam)) < 1e-13 * scale
    assert np.max(np.abs(D @ z - z * got[:, None, :])) < 1e-13 * scale
    assert np.max(np.abs(np.conj(np.swapaxes(z, 1, 2)) @ z - np.eye(nm))) < 1e-13
    # omega = sqrt(lambda) c: an error of 1e-13 of the largest lambda
    w2 = np.max(om) ** 2
    assert np.max(np.abs(om ** 2 - only ** 2)) < 2e-13 * w2


def _wide_list(s, seed):
    """The force constants on a list of 125 vectors, with small symmetric ones beyond the first
    shell and the acoustic sum rule kept."""
    import dataclasses
    nat, nm = s.n_atoms, s.n_modes
    rd = synth.box_vectors(2)
    phi = 1e-3 * np.random.default_rng(seed).standard_normal((125, nm, nm))
    row = {tuple(r): i for i, r in enumerate(rd.tolist())}
    for r, p in zip(s.rd.tolist(), s.phi_r):
        phi[row[tuple(r)]] += p
    phi = 0.5 * (phi + np.swapaxes(phi[::-1], 1, 2))
    total = phi.reshape(125, nat, 3, nat, 3).sum(axis=(0, 3))  # [s, a, b]
    for a in range(nat):
        phi[62].reshape(nat, 3, nat, 3)[a, :, a, :] -= 0.5 * (total[a] + total[a].T)
    return dataclasses.replace(s, rd=rd, phi_r=phi)


@pytest.mark.parametrize("nat,wide", [(2, False), (5, False), (5, True), (7, True)])
def test_phonon_modes_call_size(lib, nat, wide):
    """The modes of a q are the same bits alone, among 200 and among 20,000 others: near Gamma
    another order of the sum over R turns the acoustic modes into one another."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(80 + nat, n_wannier=1, n_atoms=nat, r=1)
    ds = DeviceSystem.from_host(_wide_list(s, nat) if wide else s, with_coupling=False)
    rng = np.random.default_rng(nat)
    near = np.concatenate([x * rng.standard_normal((3, 3)) for x in (1e-2, 1e-3, 1e-4, 1e-5)])
    rest = rng.uniform(-1, 1, size=(20000, 3))
    nm, out = 3 * nat, []
    for n in (0, 200, 20000):
        q = torch.from_numpy(np.concatenate([near, rest[:n]])).cuda()
        om = torch.zeros((12 + n, nm), dtype=torch.float64, device="cuda")
        z = torch.zeros((12 + n, nm, nm), dtype=torch.complex128, device="cuda")
        lib.phonon_modes(ds, q, om, z)
        out.append((om[:12].cpu().numpy(), z[:12].cpu().numpy()))
    for om, z in out[1:]:
        assert np.array_equal(om, out[0][0])
        assert np.array_equal(z, out[0][1])


@pytest.mark.parametrize("nat", range(1, 11))
def test_frequencies_alone(lib, nat):
    """omega has the same bits whether z is asked for or not, near Gamma as well."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(80 + nat, n_wannier=1, n_atoms=nat, r=1)
    ds = DeviceSystem.from_host(s, with_coupling=False)
    rng = np.random.default_rng(nat)
    q = np.concatenate([x * rng.standard_normal((20, 3)) for x in (1.0, 1e-2, 1e-4, 0.0)])
    nm = 3 * nat
    om, only = (torch.zeros((80, nm), dtype=torch.float64, device="cuda") for _ in range(2))
    z = torch.zeros((80, nm, nm), dtype=torch.complex128, device="cuda")
    lib.phonon_modes(ds, torch.from_numpy(q).cuda(), om, z)
    lib.phonon_modes(ds, torch.from_numpy(q).cuda(), only)
    assert float(om.max()) > 0
    assert torch.equal(om, only)


@pytest.mark.parametrize("nW,n_rh,npts", [
    (3, 1, 1), (5, 2, 16), (9, 3, 17), (16, 7, 33), (7, 32, 70),  # one tile a wave, K of 1 to 32
    (5, 33, 15), (9, 35, 40), (16, 66, 65), (4, 125, 1000),         # K split over waves
    (16, 1, 16390), (16, 5, 16390), (13, 34, 22000),                # four row tiles
    (32, 1, 2050), (32, 6, 2050), (32, 35, 2080),                   # two by two tiles
])
def test_fourier_sum_tiles(lib, nW, n_rh, npts):
    """Every form of the sum over lattice vectors with each remainder of its K steps, and row
    counts that leave a ragged last tile: eigenvalues of H(k)."""
    torch = torch_cuda()
    import dataclasses
    from paper_2111_14999_amd import DeviceSystem
    rng = np.random.default_rng(100 * nW + n_rh)
    s = synth.small_system(70, n_wannier=nW, n_atoms=1, r=1)
    half = synth.box_vectors(3)[172:][:n_rh // 2]  # one of every pair R, -R
    h = 0.2 * (rng.standard_normal((len(half), nW, nW)) + 1j * rng.standard_normal((len(half), nW, nW)))
    R, H = [half, -half], [h, np.conj(np.swapaxes(h, 1, 2))]
    if n_rh % 2:
        R.append(np.zeros((1, 3)))
        H.append((h[:1] + np.conj(np.swapaxes(h[:1], 1, 2))) if len(half) else np.diag(np.arange(nW))[None])
    s = dataclasses.replace(s, rh=np.concatenate(R).astype(np.int32),
                            h_r=np.concatenate(H).astype(np.complex128))
    assert len(s.rh) == n_rh
    k = rng.uniform(-1, 1, size=(npts, 3))
    eps = torch.full((npts, nW), float("nan"), dtype=torch.float64, device="cuda")
    lib.electron_bands(DeviceSystem.from_host(s, with_coupling=False), torch.from_numpy(k).cuda(), eps)
    ref = np.linalg.eigvalsh(bands.hamiltonian_k(k, s.rh, s.h_r))
    # the oracle's phases of k.R (|k.R| < 9) carry up to 1e-14 each
    assert np.max(np.abs(eps.cpu().numpy() - ref)) < 1e-12 * max(1.0, np.max(np.abs(ref)))


def test_fourier_sum_many_rows(lib):
    """32 bands at more points than two by two tiles have grid rows for."""
    torch = torch_cuda()
    import dataclasses
    from paper_2111_14999_amd import DeviceSystem, Library
    n = 32 * 65535 + 17
    s = synth.small_system(70, n_wannier=32, n_atoms=1, r=1)
    s = dataclasses.replace(s, rh=np.zeros((1, 3), dtype=np.int32), h_r=np.ascontiguousarray(s.h_r[13:14]))
    eps = torch.full((n, 32), float("nan"), dtype=torch.float64, device="cuda")
    k = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    own = Library(0)
    try:
        own.electron_bands(DeviceSystem.from_host(s, with_coupling=False), k, eps)
    finally:
        own.close()
    assert torch.equal(eps, eps[:1].expand(n, 32).contiguous())
    ref = np.linalg.eigvalsh(s.h_r[0])
    assert np.max(np.abs(eps[0].cpu().numpy() - ref)) < 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("n,npts", [(4, 1024), (4, 1025), (5, 256), (5, 257), (6, 1), (6, 1024), (7, 256),
                                    (8, 1024), (8, 1025)])
def test_eigensolver_small_batches(lib, n, npts):
    """Orders 4 to 8 on both sides of the batch at which several matrices share a wave."""
    torch = torch_cuda()
    from paper_2111_14999_amd import DeviceSystem
    s = synth.small_system(70, n_wannier=n, n_atoms=1, r=1)
    s.h_r[13] -= np.diag(np.diag(s.h_r[13])) - 0.25 * np.eye(n)
    k = np.random.default_rng(n).uniform(-1, 1, size=(npts, 3))
    eps = torch.empty((npts, n), dtype=torch.float64, device="cuda")
    U = torch.empty((npts, n, n), dtype=torch.complex128, device="cuda")
    lib.electron_bands(DeviceSystem.from_host(s, with_coupling=False), torch.from_numpy(k).cuda(), eps, U)
    eps, U = eps.cpu().numpy(), U.cpu().numpy()
    H = bands.hamiltonian_k(k, s.rh, s.h_r)
    ref = np.linalg.eigvalsh(H)
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(eps - ref)) < 1e-13 * scale
    assert np.max(np.abs(H @ U - U * eps[:, None, :])) < 1e-13 * scale
    assert np.max(np.abs(np.conj(np.swapaxes(U, 1, 2)) @ U - np.eye(n))) < 1e-13
