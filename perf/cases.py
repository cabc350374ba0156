"""The work that a program asks of this library, as cases to time and compare.

listed() holds one case of each kind of call over its real sizes, draw() another of the
same ranges; prepare() makes the inputs on the device from a seed, run() is one pass
through the public entry points, exact() the same result in plain FP64 torch and numpy.
Sizes follow the repository's own workloads: the toy CsCl crystal (6^3 mesh), the batched
crystals (4..24 Wannier functions, 2..10 atoms, meshes 16..32), the realistic perovskite
(16 Wannier functions, 15 modes, 343 lattice vectors, 40^3 mesh).
"""

from __future__ import annotations

import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2111_14999_amd import DeviceSystem, DeviceSystem3, Library

C_OMEGA = 1.054571817e-34 * math.sqrt(1.602176634e-19 / (1e-20 * 1.66053906660e-27)) / 1.602176634e-19
C_PH = 1.054571817e-34 ** 2 / (1.66053906660e-27 * 1e-20) / 1.602176634e-19
KT = 0.025851999786435535  # 300 K
SIGMA, OMEGA_MIN = 0.01, 1e-4

_handle = []


def _library():
    """A program holds one handle of the library."""
    if not _handle:
        _handle.append(Library(0))
    return _handle[0]


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # a band-structure plot: energies, phonon modes and velocities along a path
        dict(name="bands_path", kind="bands", nW=16, nat=5, r_h=3, points=301),
        # a first look at a small model: every state of a coarse mesh
        dict(name="rates_toy", kind="rates", nW=4, nat=2, r_h=1, r_g=1, n0=6, n1=6, n2=6,
             keep=0.0, prec="fp64", smearing="gaussian"),
        # a small polar crystal on an uneven mesh, odd band count
        dict(name="rates_polar", kind="rates", nW=9, nat=3, r_h=4, r_g=2, n0=24, n1=23, n2=17,
             keep=0.045, prec="fp64", smearing="gaussian", polar=True),
        # a wide band complex in the FP32 form
        dict(name="rates_wide_f32", kind="rates", nW=20, nat=5, r_h=2, r_g=2, n0=31, n1=31, n2=31,
             keep=0.032, prec="fp32", smearing="gaussian"),
        # the production calculation: full rates of the realistic crystal
        dict(name="rates_realistic", kind="rates", nW=16, nat=5, r_h=3, r_g=3, n0=40, n1=40, n2=40,
             keep=0.045, prec="fp64", smearing="gaussian"),
        # the same crystal with a width per transition
        dict(name="rates_adaptive", kind="rates", nW=16, nat=5, r_h=3, r_g=3, n0=24, n1=24, n2=24,
             keep=0.045, prec="fp64", smearing="adaptive"),
        # importance-sampled rates: weighted q lists at 64 k of the 40^3 mesh
        dict(name="rates_sampled", kind="sampled", nW=16, nat=5, r_h=3, r_g=3, n0=40, n1=40, n2=40,
             keep=0.045, nk=64, samples=4096, prec="fp64"),
        # phonon linewidths from the electron-phonon coupling
        dict(name="linewidth", kind="linewidth", nW=16, nat=5, r_h=3, r_g=3, n0=24, n1=24, n2=24,
             keep=0.045),
        # the coupling along a q path for a few k (plots, comparison with first principles)
        dict(name="interp_path", kind="interp", nW=16, nat=5, r_h=3, r_g=3, nk=4, nq=201),
        # the coupling on a full q mesh for a k of interest
        dict(name="interp_mesh", kind="interp_mesh", nW=16, nat=5, r_h=3, r_g=3, n0=24, n1=24,
             n2=24, nk=2),
        # three-phonon coupling for a few q against many q'
        dict(name="three_phonon", kind="v3", nat=5, r_v=2, nq=4, nqp=1024),
        # one optimiser step of the proposal network on a minibatch
        dict(name="train_step", kind="train", nm=15, n_harm=0, width=256, depth=4, batch=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_crystal(rng, cap):
    """nW, nat, r_h, r_g with g(Re,Rp) under `cap` bytes."""
    while True:
        c = dict(nW=rng.randint(4, 24), nat=rng.randint(2, 10), r_h=rng.randint(1, 4),
                 r_g=rng.randint(1, 3))
        if (2 * c["r_g"] + 1) ** 6 * 3 * c["nat"] * c["nW"] ** 2 * 16 <= cap:
            return c


def draw(rng):
    kind = rng.choice(["bands", "rates", "rates", "rates", "sampled", "linewidth", "interp",
                       "interp_mesh", "v3", "train"])
    if kind == "bands":
        return dict(kind=kind, nW=rng.randint(4, 24), nat=rng.randint(1, 10), r_h=rng.randint(1, 4),
                    points=_log_int(rng, 30, 3000))
    if kind in ("rates", "linewidth"):
        smearing = "adaptive" if kind == "rates" and rng.random() < 0.25 else "gaussian"
        hi = 20 if smearing == "adaptive" or kind == "linewidth" else 32
        c = dict(kind=kind, **_draw_crystal(rng, 1.5e9), n0=rng.randint(10, hi),
                 n1=rng.randint(10, hi), n2=rng.randint(10, hi), keep=rng.uniform(0.02, 0.05))
        if kind == "rates":
            c.update(smearing=smearing, prec="fp32" if smearing == "gaussian" and rng.random() < 0.35
                     else "fp64")
            c["polar"] = c["prec"] == "fp64" and rng.random() < 0.25
        return c
    if kind == "sampled":
        return dict(kind=kind, **_draw_crystal(rng, 1.5e9), n0=rng.randint(12, 32),
                    n1=rng.randint(12, 32), n2=rng.randint(12, 32), keep=0.045, nk=rng.randint(8, 64),
                    samples=_log_int(rng, 200, 4096), prec=rng.choice(["fp64", "fp64", "fp32"]))
    if kind == "interp":
        return dict(kind=kind, **_draw_crystal(rng, 1.5e9), nk=_log_int(rng, 1, 64),
                    nq=_log_int(rng, 20, 300))
    if kind == "interp_mesh":
        c = _draw_crystal(rng, 1.5e9)
        hi = max(9, min(28, int((1.5e8 / (3 * c["nat"] * c["nW"] ** 2)) ** (1 / 3))))
        return dict(kind=kind, **c, n0=rng.randint(8, hi), n1=rng.randint(8, hi),
                    n2=rng.randint(8, hi), nk=rng.randint(1, 3))
    if kind == "v3":
        nat = rng.randint(1, 6)
        return dict(kind=kind, nat=nat, r_v=rng.randint(1, 2) if nat <= 5 else 1,
                    nq=rng.randint(1, 20), nqp=_log_int(rng, 16, 1000 if nat > 3 else 3000))
    return dict(kind="train", nm=3 * rng.randint(1, 10), n_harm=rng.randint(0, 2),
                width=rng.choice([64, 96, 128, 256, 384, 512]), depth=rng.randint(2, 5),
                batch=_log_int(rng, 500, 16384))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _box(r):
    ax = np.arange(-r, r + 1, dtype=np.int32)
    return np.ascontiguousarray(np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3))


def _atoms(rng, nat):
    """Positions and the bond cutoff: CsCl, perovskite, or random positions."""
    if nat == 1:
        return np.zeros((1, 3)), 1.01
    if nat == 2:
        return np.array([[0.0, 0, 0], [0.5, 0.5, 0.5]]), 0.87
    if nat == 5:
        return np.array([[0.0, 0, 0], [0.5, 0.5, 0.5], [0.5, 0.5, 0], [0.5, 0, 0.5],
                         [0, 0.5, 0.5]]), 0.72
    while True:
        p = rng.uniform(0.0, 1.0, (nat, 3))
        d = p[:, None] - p[None]
        d -= np.round(d)
        if np.min(np.linalg.norm(d, axis=-1) + 10 * np.eye(nat)) >= 0.25:
            return p, 1.01


def _springs(rng, nat):
    """Force constants of random bond springs on R in [-1, 1]^3 (acoustic sum rule built in)."""
    pos, cutoff = _atoms(rng, nat)
    rd = _box(1)
    phi = np.zeros((27, nat, 3, nat, 3))
    for i in range(27):
        d = pos[None] + rd[i] - pos[:, None]
        dist = np.linalg.norm(d, axis=-1)
        for s, t in np.argwhere((dist < cutoff) & (dist > 1e-9)):
            if (s, t, i) > (t, s, 26 - i):  # a bond and its reverse are one
                continue
            u = d[s, t] / dist[s, t]
            K = rng.uniform(0.5, 1.5) * (0.75 * np.outer(u, u) + 0.25 * np.eye(3))
            phi[i, s, :, t] -= K
            phi[26 - i, t, :, s] -= K
            phi[13, s, :, s] += K
            phi[13, t, :, t] += K
    return rd, np.ascontiguousarray(phi.reshape(27, 3 * nat, 3 * nat))


def _hamiltonian(rng, r, nW):
    rh = _box(r)
    n = rh.shape[0]
    h = (rng.standard_normal((n, nW, nW)) + 1j * rng.standard_normal((n, nW, nW))) / math.sqrt(2.0)
    h *= np.exp(-np.linalg.norm(rh, axis=1))[:, None, None]
    for i in range(n // 2):
        h[n - 1 - i] = h[i].conj().T
    h[n // 2] = 0.5 * (h[n // 2] + h[n // 2].conj().T)
    return rh, h


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _crystal(case, seed, coupling=True):
    """(DeviceSystem, host arrays) of a random crystal with the case's sizes."""
    rng = np.random.default_rng([seed, 1])
    nW, nat, dev = case["nW"], case["nat"], _device()
    mass = rng.uniform(1.0, 3.0, nat)
    rd, phi = _springs(rng, nat)
    rh, h = _hamiltonian(rng, case["r_h"], nW)
    rg = _box(case.get("r_g", 0))
    g = None
    if coupling:
        gen = torch.Generator(device=dev).manual_seed(seed)
        n = rg.shape[0]
        g = torch.view_as_complex(torch.randn((n, n, 3 * nat, nW, nW, 2), dtype=torch.float64,
                                              device=dev, generator=gen))
        dec = torch.from_numpy(np.exp(-np.linalg.norm(rg, axis=1) / 0.8)).to(dev)
        g *= (dec / math.sqrt(2.0))[:, None, None, None, None]
        g *= dec[:, None, None, None]

    def put(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(dev)

    polar = None
    if case.get("polar"):  # charge-neutral Born charges, a dielectric tensor near 4
        Z = np.eye(3) * (rng.uniform(1.0, 3.0, nat) * (-1.0) ** np.arange(nat))[:, None, None]
        Z = Z + 0.3 * rng.standard_normal((nat, 3, 3))
        A = rng.standard_normal((3, 3))
        polar = dict(born=np.ascontiguousarray(Z - Z.mean(0)), eps_inf=4.0 * np.eye(3) + A @ A.T / 6.0,
                     alpha=5.0, g_max=3)
    ds = DeviceSystem(nW, nat, rh, put(h), rd, put(phi), put(mass), rg, rg.copy(), g, polar)
    return ds, dict(mass=mass, rd=rd, phi=phi, rh=rh, h=h, rg=rg, polar=polar)


def _mesh(case):
    return case["n0"], case["n1"], case["n2"]


def _mesh_points(mesh, idx=None):
    idx = np.arange(mesh[0] * mesh[1] * mesh[2]) if idx is None else np.asarray(idx, dtype=np.int64)
    return np.stack([idx // (mesh[1] * mesh[2]) / mesh[0], idx // mesh[2] % mesh[1] / mesh[1],
                     idx % mesh[2] / mesh[2]], axis=1)


def _threads(f, n, size=2048):
    """f(slice) over chunks of n rows on the host's cores, concatenated."""
    with ThreadPoolExecutor(min(16, os.cpu_count() or 1)) as ex:
        parts = list(ex.map(f, [slice(a, min(n, a + size)) for a in range(0, n, size)]))
    return [np.concatenate(p) for p in zip(*parts)]


def _eig(pts, r, m, vectors=True):
    """Eigenvalues (and vectors) of sum_R e^{i 2 pi x.R} m(R) at the points."""
    flat = m.reshape(m.shape[0], -1)

    def one(sl):
        a = (np.exp(2j * np.pi * (pts[sl] @ r.T.astype(float))) @ flat).reshape(-1, *m.shape[1:])
        a = 0.5 * (a + np.conj(np.swapaxes(a, 1, 2)))
        return np.linalg.eigh(a) if vectors else (np.linalg.eigvalsh(a),)

    return _threads(one, pts.shape[0], 256)


def _window(case, host, seed):
    """Chemical potential near the band bottom such that about `keep` of the mesh's k have a
    state within 0.3 eV of it (from a sample of mesh points), and sampled k in the window."""
    rng = np.random.default_rng([seed, 2])
    mesh = _mesh(case)
    N = mesh[0] * mesh[1] * mesh[2]
    idx = rng.permutation(N)[:4096]
    e0 = _eig(_mesh_points(mesh, idx), host["rh"], host["h"], vectors=False)[0][:, 0]
    order = np.sort(e0)
    i = min(len(order) - 2, max(8, int(case["keep"] * len(order))))
    mu = float(0.5 * (order[i] + order[i + 1])) - 0.3  # the edge between two sampled energies
    return mu, idx[np.abs(e0 - mu) < 0.299]


def _params(case, mu):
    if case.get("keep", 0.0) == 0.0:  # every state
        return dict(mu=mu, kT=KT, sigma=0.02, win_lo=-1e30, win_hi=1e30, omega_min=OMEGA_MIN)
    p = dict(mu=mu, kT=KT, sigma=SIGMA, win_lo=mu - 0.3, win_hi=mu + 0.3, omega_min=OMEGA_MIN)
    if case.get("smearing") == "adaptive":
        p.update(smearing="adaptive", adaptive_scale=1.0)
    return p


def _q_path(rng, n):
    """n points along segments between corners of the cell, none of them a corner."""
    c = np.array([[0, 0, 0], [0.5, 0, 0], [0.5, 0.5, 0], [0, 0, 0], [0.5, 0.5, 0.5], [0.5, 0, 0]])
    t = (np.arange(n) + rng.uniform(0.3, 0.7)) / n * 5
    i = np.minimum(t.astype(int), 4)
    return c[i] + (t - i)[:, None] * (c[i + 1] - c[i])


def _features(case, rng):
    nm, nh, B = case["nm"], case["n_harm"], case["batch"]
    kq = rng.integers(0, 40, (B, 6)) / 40.0
    e = rng.uniform(-1, 1, (B, 1))
    hot = np.eye(nm)[rng.integers(0, nm, B)]
    if nh == 0:
        return np.concatenate([kq[:, :3], e, kq[:, 3:], hot], axis=1)
    cols = [e, hot]
    for h in range(1, nh + 1):
        cols.append(np.stack([np.cos(2 * np.pi * h * kq), np.sin(2 * np.pi * h * kq)], -1).reshape(B, 12))
    return np.concatenate(cols, axis=1)


def _layers(case):
    n_in = 7 + case["nm"] if case["n_harm"] == 0 else 1 + case["nm"] + 12 * case["n_harm"]
    widths = [n_in] + [case["width"]] * case["depth"] + [1]
    return n_in, list(zip(widths[1:], widths[:-1]))


def _train_inputs(case, seed):
    rng = np.random.default_rng([seed, 3])
    X = _features(case, rng).astype(np.float32)
    y = (rng.normal(-4.0, 1.3, case["batch"])).astype(np.float32)
    _, shapes = _layers(case)
    theta = np.concatenate([np.concatenate([rng.uniform(-1, 1, o * i) / math.sqrt(i),
                                            rng.normal(0, 0.02, o)]) for o, i in shapes])
    # moments of a run in progress
    m1 = rng.normal(0, 1e-3, theta.size)
    m2 = rng.uniform(0.5, 2.0, theta.size) * 1e-4
    return X, y, theta.astype(np.float32), m1.astype(np.float32), m2.astype(np.float32)


def _v3_inputs(case, seed):
    rng = np.random.default_rng([seed, 4])
    dev, nm = _device(), 3 * case["nat"]
    mass = rng.uniform(1.0, 3.0, case["nat"])
    rd, phi = _springs(rng, case["nat"])
    r = _box(case["r_v"])
    gen = torch.Generator(device=dev).manual_seed(seed)
    phi3 = torch.randn((r.shape[0], r.shape[0], nm, nm, nm), dtype=torch.float64, device=dev,
                       generator=gen)
    dec = torch.from_numpy(np.exp(-np.linalg.norm(r, axis=1) / 0.8)).to(dev)
    phi3 *= dec[:, None, None, None, None] * dec[:, None, None, None]
    put = torch.from_numpy
    s3 = DeviceSystem3(case["nat"], rd, put(phi).to(dev), put(mass).to(dev), r, r.copy(), phi3)
    q = put(rng.uniform(-1, 1, (case["nq"], 3))).to(dev)
    qp = put(rng.uniform(-1, 1, (case["nqp"], 3))).to(dev)
    return s3, q, qp


def prepare(case, seed):
    lib, dev, kind = _library(), _device(), case["kind"]
    st = dict(case=case, lib=lib)

    def zeros(*shape, dtype=torch.float64):
        return torch.zeros(shape, dtype=dtype, device=dev)

    if kind == "train":
        X, y, theta, m1, m2 = (torch.from_numpy(a).to(dev) for a in _train_inputs(case, seed))
        st.update(X=X, y=y, theta=theta, m1=m1, m2=m2, grad=torch.zeros_like(theta), step=500)
        return st
    if kind == "v3":
        s3, q, qp = _v3_inputs(case, seed)
        nm = 3 * case["nat"]
        st.update(s3=s3, q=q, qp=qp,
                  out=zeros(case["nq"], case["nqp"], nm, nm, nm, dtype=torch.complex128))
        return st
    rng = np.random.default_rng([seed, 5])
    ds, host = _crystal(case, seed, coupling=kind != "bands")
    st["ds"] = ds
    nW, nm = case["nW"], 3 * case["nat"]
    if kind == "bands":
        n = case["points"]
        st.update(k=torch.from_numpy(_q_path(rng, n)).to(dev), eps=zeros(n, nW), om=zeros(n, nm),
                  v=zeros(n, nW, 3))
        return st
    if kind == "interp":
        nk, nq = case["nk"], case["nq"]
        st.update(k=torch.from_numpy(rng.uniform(0, 1, (nk, 3))).to(dev),
                  q=torch.from_numpy(_q_path(rng, nq)).to(dev),
                  g=zeros(nk, nq, nm, nW, nW, dtype=torch.complex128), ek=zeros(nk, nW),
                  ekq=zeros(nk, nq, nW), om=zeros(nq, nm))
        return st
    mesh = _mesh(case)
    N = mesh[0] * mesh[1] * mesh[2]
    st["mesh"] = mesh
    if kind == "interp_mesh":
        nk = case["nk"]
        k = _mesh_points(mesh, rng.integers(0, N, nk))
        st.update(k=torch.from_numpy(k).to(dev), ek=zeros(nk, nW), ekq=zeros(nk, N, nW),
                  g=zeros(nk, N, nm, nW, nW, dtype=torch.complex128))
        return st
    mu, inside = _window(case, host, seed)
    st["par"] = _params(case, mu)
    if kind == "linewidth":
        st.update(P=zeros(N, nm), gamma=zeros(N, nW))
    elif kind == "sampled":
        nk, S = case["nk"], case["samples"]
        kidx = np.sort(np.resize(inside, nk)).astype(np.int32)
        w = rng.uniform(0.5, 1.5, nk * S) / S
        st.update(k=torch.from_numpy(kidx).to(dev), gamma=zeros(nk, nW),
                  q=(torch.arange(0, nk * S + 1, S, dtype=torch.int64, device=dev),
                     torch.from_numpy(rng.integers(0, N, nk * S).astype(np.int32)).to(dev),
                     torch.from_numpy(w).to(dev)))
    else:
        st.update(gamma=zeros(N, nW), mask=zeros(N, nW, dtype=torch.uint8),
                  kept=zeros(N, dtype=torch.int32))
    return st


def run(st):
    lib, case = st["lib"], st["case"]
    kind = case["kind"]
    if kind == "rates":
        n = lib.scatter_rates(st["ds"], st["mesh"], st["par"], st["gamma"], precision=case["prec"],
                              band_mask=st["mask"], kept_k_out=st["kept"])
        # (rows of the first n kept k; the rest of the buffers is not written)
        return dict(n_kept=n, gamma=st["gamma"], mask=st["mask"], kept=st["kept"])
    if kind == "sampled":
        n = lib.scatter_rates(st["ds"], st["mesh"], st["par"], st["gamma"], k_idx=st["k"],
                              q_lists=st["q"], precision=case["prec"])
        return dict(n_kept=n, gamma=st["gamma"])
    if kind == "linewidth":
        n = lib.phonon_linewidth(st["ds"], st["mesh"], st["par"], st["P"], gamma_out=st["gamma"])
        return dict(n_kept=n, P=st["P"], gamma=st["gamma"])
    if kind == "interp":
        lib.interp_g(st["ds"], st["k"], st["q"], st["g"], eps_k=st["ek"], eps_kq=st["ekq"],
                     omega_q=st["om"])
        return dict(g=st["g"], eps_k=st["ek"], eps_kq=st["ekq"], omega_q=st["om"])
    if kind == "interp_mesh":
        lib.interp_g_mesh(st["ds"], st["k"], st["mesh"], st["g"], eps_k=st["ek"], eps_kq=st["ekq"])
        return dict(g=st["g"], eps_k=st["ek"], eps_kq=st["ekq"])
    if kind == "bands":
        lib.electron_bands(st["ds"], st["k"], st["eps"])
        lib.phonon_modes(st["ds"], st["k"], st["om"])
        lib.velocities(st["ds"], st["k"], st["v"])
        return dict(eps=st["eps"], omega=st["om"], v=st["v"])
    if kind == "v3":
        lib.interp_v3(st["s3"], st["q"], st["qp"], st["out"])
        return dict(v3=st["out"])
    n_in, _ = _layers(case)
    loss = lib.mlp_grad(st["theta"], st["X"], st["y"], st["grad"], n_in, case["width"], case["depth"])
    st["step"] += 1
    lib.mlp_adam(st["theta"], st["grad"], st["m1"], st["m2"], st["step"], 3e-4)
    return dict(loss=loss, grad=st["grad"], theta=st["theta"], m1=st["m1"], m2=st["m2"])


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "train":
        n_in, shapes = _layers(case)
        p, B = sum(o * i + o for o, i in shapes), case["batch"]
        return dict(bytes=4.0 * (B * (n_in + 1) + 8 * p),
                    flops=2.0 * B * sum(o * i for o, i in shapes) * 3 - 2.0 * B * shapes[0][0] * n_in)
    nm = 3 * case["nat"]
    if kind == "v3":
        n = (2 * case["r_v"] + 1) ** 3
        pairs, m3 = case["nq"] * case["nqp"], nm ** 3
        return dict(bytes=8.0 * n * n * m3 + 16.0 * pairs * m3,
                    flops=4.0 * case["nq"] * n * n * m3 + 8.0 * pairs * m3 * (n + 2 * nm))
    nW = case["nW"]
    nrh = (2 * case["r_h"] + 1) ** 3
    eig = 8.0 * (nrh * nW ** 2 + 9 * nW ** 3) + 4.0 * 27 * nm ** 2 + 72.0 * nm ** 3  # a point's tables
    if kind == "bands":
        n = case["points"]
        return dict(bytes=16.0 * nrh * nW ** 2 + n * (24 + 8 * nm + 32 * nW),
                    flops=n * (eig + 24.0 * nW ** 2 * (nrh + nW + 1)))
    W = 2 * case["r_g"] + 1
    cols, g_bytes = nm * nW, 16.0 * W ** 6 * nm * nW ** 2
    rot = 8.0 * nm * nW * (nm + nW)  # one band n: U_{k+q} and z of one (k, q)
    if kind == "interp":
        nk, nq = case["nk"], case["nq"]
        return dict(bytes=g_bytes + 16.0 * nk * nq * cols * nW,
                    flops=8.0 * nk * W ** 3 * cols * nW * (W ** 3 + nW) +
                    nk * nq * (8.0 * W ** 3 * cols * nW + nW * rot + eig))
    N = case["n0"] * case["n1"] * case["n2"]
    n12 = case["n1"] * case["n2"]
    axes = 8.0 * (W ** 3 * case["n2"] + W ** 2 * n12 + W * N)  # Rp sum of one column, axis by axis
    if kind == "interp_mesh":
        nk = case["nk"]
        return dict(bytes=g_bytes + 16.0 * nk * N * cols * nW,
                    flops=8.0 * nk * W ** 3 * cols * nW * (W ** 3 + nW) +
                    nk * nW * (axes * cols + N * rot) + N * eig)
    if kind == "sampled":
        nk, S = case["nk"], case["samples"]
        return dict(bytes=g_bytes + nk * S * 12.0,
                    flops=8.0 * nk * W ** 3 * cols * (W ** 3 * nW + nW) +
                    nk * S * (8.0 * W ** 3 * cols + 8.0 * cols + 8.0 * nm * nm) + N * eig)
    states = N * (case["keep"] or float(nW))
    live = 0.2 if case["keep"] else 1.0  # of the (k, q) pairs, a final state in reach
    if case.get("smearing") == "adaptive":
        live = 1.0
    per = axes * cols + N * (8.0 * cols + 8.0 * nm * nm)
    return dict(bytes=g_bytes + states * 8.0 * nW,
                flops=N * eig + states * (live * per + 8.0 * W ** 3 * cols * nW * (W + 1)))


# ----------------------------------------------------------------------------
# the same in plain FP64
# ----------------------------------------------------------------------------

def _phonons(pts, host):
    m = np.repeat(host["mass"], 3)
    lam, z = _eig(pts, host["rd"], host["phi"] / np.sqrt(m[:, None] * m[None]))
    om = C_OMEGA * np.sqrt(np.maximum(lam, 0.0))
    act = om >= OMEGA_MIN
    l = np.where(act[:, None, :], np.sqrt(C_PH / (2.0 * m[None, :, None] *
                                                  np.where(act, om, 1.0)[:, None, :])), 0.0)
    nb = np.where(act, 1.0 / np.expm1(np.where(act, om, 1.0) / KT), 0.0)
    return om, z * l, nb, act


def _velocities(pts, host, U):
    """Diagonal group velocities (the random crystals' bands are not degenerate)."""
    flat = host["h"].reshape(host["h"].shape[0], -1)
    r = host["rh"].astype(float)
    nW = U.shape[1]

    def one(sl):
        ph = np.exp(2j * np.pi * (pts[sl] @ r.T))
        out = np.empty((ph.shape[0], nW, 3))
        for a in range(3):
            d = ((ph * (1j * r[:, a])) @ flat).reshape(-1, nW, nW)
            out[:, :, a] = np.sum(np.conj(U[sl]) * (d @ U[sl]), axis=1).real
        return (out,)

    return _threads(one, pts.shape[0], 256)[0]


def _polar_factor(pts, host, zl):
    """L(q, nu) of the long-range coupling i L(q, nu) [U_k^+ U_{k+q}]."""
    p, D = host["polar"], np.zeros((len(pts), 3 * len(host["mass"])))
    for G in _box(p["g_max"]):
        K = 2 * np.pi * (pts + G)
        den = np.einsum("qa,ab,qb->q", K, p["eps_inf"], K)
        ok = np.linalg.norm(K, axis=1) > 1e-12
        w = np.where(ok, np.exp(-den / (4 * p["alpha"])) / np.where(ok, den, 1.0), 0.0)
        D += w[:, None] * np.einsum("qa,sab->qsb", K, p["born"]).reshape(D.shape)
    e2 = 1.602176634e-19 / (4 * np.pi * 8.8541878128e-12 * 1e-10)
    return 4 * np.pi * e2 * np.einsum("qs,qsv->qv", D, zl)


def _exact_rates(case, seed):
    kind, mesh, dev = case["kind"], _mesh(case), _device()
    nW, nm = case["nW"], 3 * case["nat"]
    N = mesh[0] * mesh[1] * mesh[2]
    states = N * (case["keep"] or float(nW)) if kind != "sampled" else 1.1 * case["nk"]
    if states * nm * nW * (N if kind != "sampled" else case["samples"]) > 5e10:
        return None  # over about 20 seconds
    st = prepare(case, seed)
    _, host = _crystal(case, seed, coupling=False)
    p, g = st["par"], st["ds"].g_rr
    pts = _mesh_points(mesh)
    eps, U = _eig(pts, host["rh"], host["h"])
    om, zl, nb, act = _phonons(pts, host)
    v = _velocities(pts, host, U) if p.get("smearing") == "adaptive" else None
    mask = (eps > p["win_lo"]) & (eps < p["win_hi"])
    kept = st["k"].cpu().numpy() if kind == "sampled" else np.nonzero(mask.any(1))[0]
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    teps, tU, tE, tom, tnb = put(eps), put(U), put(np.swapaxes(zl, 1, 2)), put(om), put(nb)
    x = (teps - p["mu"]) / KT
    tf = 1.0 / (1.0 + torch.exp(x))
    tact, tpts = put(act), put(pts)
    tL = put(_polar_factor(pts, host, zl)) if host["polar"] else None
    rg = put(host["rg"].astype(float))
    tv = put(v) if v is not None else None
    steps = put(2.0 * np.pi / np.asarray(mesh, dtype=float)) / math.sqrt(12.0)
    gamma = np.zeros((len(kept) if kind == "sampled" else N, nW))
    P = torch.zeros((N, nm), dtype=torch.float64, device=dev)
    tri = np.stack([np.arange(N) // (mesh[1] * mesh[2]), np.arange(N) // mesh[2] % mesh[1],
                    np.arange(N) % mesh[2]])
    ttri = put(tri)
    phase = torch.exp(2j * math.pi * (tpts @ rg.T)) if kind != "sampled" else None  # [N, Rp]
    g2d = g.reshape(g.shape[0], -1)
    for b0 in range(0, len(kept), 16):
        rows = kept[b0:b0 + 16]
        pk = torch.exp(2j * math.pi * (put(pts[rows]) @ rg.T))
        G = (pk @ g2d).reshape((len(rows),) + tuple(g.shape[1:]))
        for j, ik in enumerate(rows):
            a = b0 + j
            if kind == "sampled":
                q = st["q"][1][a * case["samples"]:(a + 1) * case["samples"]].long()
                wq = st["q"][2][a * case["samples"]:(a + 1) * case["samples"]]
                ph = torch.exp(2j * math.pi * (tpts[q] @ rg.T))
            else:
                q, wq, ph = torch.arange(N, device=dev), None, phase
            s = [(ttri[d][q] + int(tri[d, ik])) % mesh[d] for d in range(3)]
            kq = (s[0] * mesh[1] + s[1]) * mesh[2] + s[2]
            for n in np.nonzero(mask[ik])[0]:
                F = (G[j] * torch.conj(tU[ik, :, n])[None, None, :, None]).sum(2)  # [Rp, sa, b]
                X = (ph @ F.reshape(F.shape[0], -1)).reshape(-1, nm, nW)
                gq = torch.bmm(tE[q], torch.bmm(X, tU[kq]))  # [q, nu, m]
                if tL is not None:
                    O = (torch.conj(tU[ik, :, n])[None, :, None] * tU[kq]).sum(1)
                    gq += 1j * tL[q][:, :, None] * O[:, None, :]
                g2 = gq.abs().square()
                en = teps[ik, n]
                d = (en - teps[kq])[:, None, :]
                sg = torch.tensor(p["sigma"], dtype=torch.float64, device=dev)
                if tv is not None:
                    sg = torch.sqrt((((tv[ik, n] - tv[kq]) * steps) ** 2).sum(-1))[:, None, :]
                    sg = torch.clamp(sg, min=p["sigma"])
                w, bn, fm = tom[q][:, :, None], tnb[q][:, :, None], tf[kq][:, None, :]
                em = torch.exp(-((d - w) / sg) ** 2) / (math.sqrt(math.pi) * sg)
                ab = torch.exp(-((d + w) / sg) ** 2) / (math.sqrt(math.pi) * sg)
                if kind == "linewidth":
                    P += tf[ik, n] * (1 - tf[ik, n]) / KT * (g2 * em).sum(2)
                t = (g2 * ((bn + 1 - fm) * em + (bn + fm) * ab)).sum(2) * tact[q]
                t = t.sum(1)
                gamma[a, n] = 2 * math.pi * float((t * wq).sum() if wq is not None else t.sum() / N)
    if kind == "sampled":
        return dict(n_kept=None, gamma=gamma)
    if kind == "linewidth":
        P = torch.where(tact, 2 * math.pi / N * tnb * (tnb + 1) * tom * P, torch.zeros_like(P))
        return dict(n_kept=None, P=P.cpu().numpy(), gamma=gamma)
    return dict(n_kept=None, gamma=gamma, mask=None, kept=None)


def _exact_train(case, seed):
    X, y, theta, m1, m2 = (a.astype(np.float64) for a in _train_inputs(case, seed))
    _, shapes = _layers(case)
    acts, zs, off, Ws = [X], [], 0, []
    for o, i in shapes:
        W, b = theta[off:off + o * i].reshape(o, i), theta[off + o * i:off + o * i + o]
        Ws.append((off, W))
        off += o * i + o
        zs.append(acts[-1] @ W.T + b)
        acts.append(zs[-1] / (1.0 + np.exp(-zs[-1])))
    r = zs[-1][:, 0] - y
    grad = np.zeros_like(theta)
    d = (2.0 * r / len(y))[:, None]
    for l in range(len(shapes) - 1, -1, -1):
        (off, W), (o, i) = Ws[l], shapes[l]
        grad[off:off + o * i] = (d.T @ acts[l]).ravel()
        grad[off + o * i:off + o * i + o] = d.sum(0)
        if l:
            s = 1.0 / (1.0 + np.exp(-zs[l - 1]))
            d = (d @ W) * s * (1.0 + zs[l - 1] * (1.0 - s))
    m1 = 0.9 * m1 + 0.1 * grad
    m2 = 0.999 * m2 + 0.001 * grad ** 2
    t = 501
    theta = theta - 3e-4 * (m1 / (1 - 0.9 ** t)) / (np.sqrt(m2 / (1 - 0.999 ** t)) + 1e-8)
    return dict(loss=float(np.mean(r ** 2)), grad=grad, theta=theta, m1=m1, m2=m2)


def exact(case, seed):
    """run()'s outputs in FP64; eigenvector phases leave g and V3 without a value of their own."""
    kind = case["kind"]
    if kind in ("rates", "sampled", "linewidth"):
        return _exact_rates(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "v3":
        return None
    _, host = _crystal(case, seed, coupling=False)
    rng = np.random.default_rng([seed, 5])
    if kind == "bands":
        k = _q_path(rng, case["points"])
        eps, U = _eig(k, host["rh"], host["h"])
        return dict(eps=eps, omega=_phonons(k, host)[0], v=_velocities(k, host, U))
    if kind == "interp":
        k, q = rng.uniform(0, 1, (case["nk"], 3)), None
        q = _q_path(rng, case["nq"])
    else:
        mesh = _mesh(case)
        q = _mesh_points(mesh)
        k = _mesh_points(mesh, rng.integers(0, len(q), case["nk"]))
    kq = (k[:, None] + q[None]).reshape(-1, 3)
    out = dict(g=None, eps_k=_eig(k, host["rh"], host["h"], False)[0],
               eps_kq=_eig(kq, host["rh"], host["h"], False)[0].reshape(len(k), len(q), -1))
    if kind == "interp":
        out["omega_q"] = _phonons(q, host)[0]
    return out
