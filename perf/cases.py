"""Timed cases of the real-time TDDFT path, each through the public entry points.

A case is a plain dict; its "kind" says which call a pass makes:

  apply     Grid.apply_h for every k-point (one H.psi of resident states)
  etrs      Grid.propagate_etrs over a few steps, with norms (and the dipole on
            a finite grid), the states advancing in place
  cfm4      the same with Grid.propagate_cfm4
  batch     Batch.step: one ETRS step of several resident jobs (serving)
  observe   what a run prints between propagations: density, norms, Gram
            matrix, current, energy (and dipole / Hartree potential)
  spectrum  strength function and conductivity of recorded traces

Inputs are made from the seed alone: atoms at random places, smooth random
orthonormal states (Fourier modes up to 3, Bloch phases on periodic axes, a
Gaussian envelope on finite ones) and the potential of smeared ions.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1912_07921_amd import ks, serving
from paper_1912_07921_amd import workloads as W

RLOC = 0.5                                  # width of the smeared ions (bohr)
LASER = (0.05, 0.057, 20.0 * W.FS_AU, 0.0, 0.0, 1.0)
T_LASER = 100.0                             # a time inside the pulse
MMAX = 3
C_LAP = (-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0)
C_GRAD = (0.0, 4.0 / 5.0, -1.0 / 5.0, 4.0 / 105.0, -1.0 / 280.0)


def _system(kind, n, per, nk, ns, natoms, lmax, **kw):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], h=0.2, per=per, nk=nk,
             ns=ns, natoms=natoms, lmax=lmax, laser=False, hartree=False,
             mixed=False, autotune=False, nsteps=1, dt=0.005)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest request of the serving mix, H applied once: latency
        # and launches
        dict(_system("apply", (24, 24, 24), "000", 1, 4, 2, 1),
             name="apply_small"),
        # a crystal cell of odd sizes with two k-points, inside the laser
        # pulse: Bloch phases, the gradient term, ragged tiles
        dict(_system("apply", (45, 50, 39), "111", 2, 13, 11, 2, h=0.3,
                     laser=True), name="apply_ragged_crystal"),
        # the large grid in mixed precision, a quarter of its states (a
        # caller that works through them in groups)
        dict(_system("apply", (128, 128, 128), "000", 1, 64, 64, 2, h=0.18,
                     mixed=True), name="apply_large_mixed"),
        # a small molecule with the Hartree term: many short launches
        dict(_system("etrs", (24, 24, 24), "000", 1, 4, 2, 1, hartree=True,
                     nsteps=10, dt=0.01), name="etrs_small_hartree"),
        # the ordinary molecule: 64^3, 32 states, 8 atoms with s and p
        dict(_system("etrs", (64, 64, 64), "000", 1, 32, 8, 1, nsteps=4),
             name="etrs_molecule"),
        dict(_system("etrs", (64, 64, 64), "000", 1, 32, 8, 1, nsteps=4,
                     mixed=True), name="etrs_molecule_mixed"),
        # the laser-driven crystal: 48^3, 4 k-points of 64 states, in the
        # shape the library's tuner picks
        dict(_system("etrs", (48, 48, 48), "111", 4, 64, 16, 1, h=0.3,
                     laser=True, autotune=True, nsteps=2, dt=0.02),
             name="etrs_crystal"),
        # the other propagator, with the Hartree term, on a box whose sides
        # differ
        dict(_system("cfm4", (72, 60, 66), "000", 1, 40, 10, 1, hartree=True,
                     nsteps=2), name="cfm4_ragged_hartree"),
        # the largest: 128^3, 256 states, 64 atoms with s, p and d
        dict(_system("etrs", (128, 128, 128), "000", 1, 256, 64, 2, h=0.18),
             name="etrs_large"),
        # a serving step: resident requests of mixed sizes
        dict(kind="batch", njobs=16, mix=4, mixed=False, name="batch_serving"),
        # the observables of the crystal between propagations
        dict(_system("observe", (48, 48, 48), "111", 4, 64, 16, 1, h=0.3,
                     laser=True), name="observe_crystal"),
        # after the run: spectra of a full-length trace
        dict(kind="spectrum", nt=501, nw=2000, dt=0.005, name="spectrum"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fft_size(n):
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


def draw(rng):
    """One more case: every kind, sizes spread over their logarithm."""
    kind = rng.choice(["apply", "apply", "etrs", "etrs", "cfm4", "batch",
                       "observe", "spectrum"])
    if kind == "spectrum":
        return dict(kind=kind, nt=_log_int(rng, 101, 2001),
                    nw=_log_int(rng, 200, 4000), dt=0.005)
    if kind == "batch":
        return dict(kind=kind, njobs=_log_int(rng, 2, 24),
                    mix=rng.randrange(1000), mixed=rng.random() < 0.4)
    per = rng.choice(["000", "000", "111", "111", "110"])
    h = rng.choice([0.18, 0.2, 0.25, 0.3])
    if per != "000":
        h = max(h, 0.25)
    base = _log_int(rng, 24, 112)
    n = [max(20, min(128, int(base * rng.uniform(0.75, 1.25))))
         for _ in range(3)]
    hartree = kind != "apply" and per != "110" and rng.random() < 0.4
    if hartree and per == "111":
        n = [_fft_size(v) for v in n]
    nk = 1 if per == "000" else rng.choice([1, 2, 4])
    most = 0.25 * 128 ** 3 * 256            # points x states x steps
    steps = 1 if kind in ("apply", "observe") else rng.choice([1, 2, 3])
    room = int(most / (n[0] * n[1] * n[2] * nk * steps))
    return _system(kind, n, per, nk, max(1, min(_log_int(rng, 2, 96), room)),
                   _log_int(rng, 1, 40), rng.choice([0, 1, 1, 2]), h=h,
                   laser=per != "000" or rng.random() < 0.2, hartree=hartree,
                   mixed=kind != "observe" and rng.random() < 0.4,
                   autotune=kind in ("etrs", "cfm4") and rng.random() < 0.3,
                   nsteps=steps, dt=0.01 if h >= 0.25 else 0.005)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _axis(n, h, per):
    i = np.arange(n, dtype=np.float64)
    return i * h if per else (i - 0.5 * (n - 1)) * h


def _describe(case, seed):
    """The system as plain numbers: grid, k-points, atoms, projectors."""
    r = np.random.Generator(np.random.PCG64(seed))
    n = (case["nx"], case["ny"], case["nz"])
    h = (case["h"],) * 3
    per = tuple(int(ch) for ch in case["per"])
    L = np.array([n[a] * h[a] for a in range(3)])
    nk, na = case["nk"], case["natoms"]
    signs = np.array([[1, 1, 0], [1, -1, 0], [-1, 1, 0], [-1, -1, 0]])
    kpts = (0.25 * 2 * np.pi / L) * signs[:nk] * np.array(per)
    # in a cell: anywhere; in a box: a ball well inside
    ball = r.standard_normal((na, 3))
    ball *= (0.3 * L.min() * r.uniform(0, 1, (na, 1)) ** (1 / 3)
             / np.linalg.norm(ball, axis=1, keepdims=True))
    cell = r.uniform(0, 1, (na, 3)) * L
    pos = np.where(np.array(per)[None, :] == 1, cell, ball)
    rc = 2.5 if case["lmax"] == 2 else 2.0
    rc = min([rc] + [0.45 * L[a] for a in range(3) if per[a]])
    return dict(n=n, h=h, per=per, kpts=kpts, kw=np.full(nk, 1.0 / nk),
                ns=case["ns"], occ=np.full(case["ns"], 2.0), pos=pos,
                Z=r.choice(np.array([1.0, 4.0, 6.0]), na),
                lmax=case["lmax"], rc=rc, sigma=rc / 4,
                E=r.uniform(-2.0, 2.0, (na, 3)), xc=1,
                laser=LASER if case["laser"] else (0, 0, 0, 0, 0, 1.0),
                hartree=int(case["hartree"]))


def _vion(d, dev):
    """Potential of the smeared ions; by Fourier sum when an axis is
    periodic."""
    n, h, per = d["n"], d["h"], d["per"]
    X = [torch.from_numpy(_axis(n[a], h[a], per[a])).to(dev)
         for a in range(3)]
    if not any(per):
        v = torch.zeros(n[2], n[1], n[0], dtype=torch.float64, device=dev)
        for p, Z in zip(d["pos"], d["Z"]):
            q = torch.sqrt((X[2][:, None, None] - p[2]) ** 2
                           + (X[1][None, :, None] - p[1]) ** 2
                           + (X[0][None, None, :] - p[0]) ** 2)
            q = q.clamp_min(1e-9)
            v -= Z * torch.special.erf(q / RLOC) / q
        return v.reshape(-1)
    g = [2 * np.pi * torch.fft.fftfreq(n[a], d=h[a], dtype=torch.float64,
                                       device=dev) for a in range(3)]
    G2 = (g[2][:, None, None] ** 2 + g[1][None, :, None] ** 2
          + g[0][None, None, :] ** 2)
    S = torch.zeros(n[2], n[1], n[0], dtype=torch.complex128, device=dev)
    for p, Z in zip(d["pos"], d["Z"]):
        e = [torch.exp(-1j * g[a] * (p[a] - float(X[a][0])))
             for a in range(3)]
        S -= Z * e[2][:, None, None] * e[1][None, :, None] * e[0]
    vol = h[0] * h[1] * h[2]
    S *= 4 * np.pi * torch.exp(-G2 * RLOC ** 2 / 4) / vol
    S /= torch.where(G2 > 0, G2, torch.ones_like(G2))
    S[0, 0, 0] = 0.0
    return torch.fft.ifftn(S).real.contiguous().reshape(-1)


def _states(d, seed, dev):
    """[nk, ns, N] smooth random states, orthonormal within each k-point."""
    n, h, per, ns = d["n"], d["h"], d["per"], d["ns"]
    N = n[0] * n[1] * n[2]
    r = np.random.Generator(np.random.PCG64([seed, 1]))
    ms = torch.arange(-MMAX, MMAX + 1, dtype=torch.float64, device=dev)
    nm = len(ms)
    out = torch.empty(len(d["kw"]), ns, N, dtype=torch.complex128, device=dev)
    for k, kp in enumerate(d["kpts"]):
        f = []
        for a in range(3):
            x = torch.from_numpy(_axis(n[a], h[a], per[a])).to(dev)
            L = n[a] * h[a]
            e = torch.exp(2j * np.pi * torch.outer(ms, x) / L)
            w = L / 4
            e = e * (torch.exp(1j * kp[a] * x) if per[a]
                     else torch.exp(-x * x / (2 * w * w)))
            f.append(e)
        c = r.standard_normal((ns, nm, nm, nm, 2)) @ np.array([1, 1j])
        t = torch.from_numpy(c).to(dev)
        t = torch.tensordot(t, f[2], dims=([3], [0]))       # s, x, y, Z
        t = torch.tensordot(t, f[1], dims=([2], [0]))       # s, x, Z, Y
        t = torch.tensordot(t, f[0], dims=([1], [0]))       # s, Z, Y, X
        psi = t.reshape(ns, N)
        S = ((psi @ psi.conj().T) * (h[0] * h[1] * h[2])).cpu().numpy()
        inv = np.linalg.inv(np.linalg.cholesky(S))
        torch.matmul(torch.from_numpy(inv).to(dev), psi, out=out[k])
        del t, psi
    return out


def _spec(d):
    na = len(d["Z"])
    return W.SystemSpec(n=d["n"], h=d["h"], periodic=d["per"],
                        kpts=d["kpts"], kw=d["kw"], nstates=d["ns"],
                        occ=d["occ"], pos=d["pos"], Z=d["Z"],
                        lmax=np.full(na, d["lmax"]), rc=np.full(na, d["rc"]),
                        sigma=np.full(na, d["sigma"]), E=d["E"], xc=d["xc"],
                        laser=d["laser"], hartree=d["hartree"])


def _requests(case):
    """The resident requests of a batch: sizes of the serving mix."""
    r = random.Random(case["mix"])
    return [_system("etrs", (n, n, n), "000", 1, ns, na, 1)
            for n, ns, na in ((r.choice([24, 32, 48, 64, 80]),
                               r.choice([4, 8, 16, 32, 64]),
                               r.randint(2, 12))
                              for _ in range(case["njobs"]))]


def _trace(case, seed):
    """Dipole trace of a kicked run and a current trace: damped sums of
    oscillations, [nt, 3]."""
    r = np.random.Generator(np.random.PCG64(seed))
    t = np.arange(case["nt"]) * case["dt"]
    out = []
    for _ in range(2):
        om = r.uniform(0.1, 3.0, (12, 3))
        am = 0.01 * r.standard_normal((12, 3))
        ph = r.uniform(0, 2 * np.pi, (12, 3))
        f = (am * np.sin(om * t[:, None, None] + ph)).sum(1)
        out.append(f * np.exp(-0.02 * t)[:, None])
    return out[0], out[1], np.linspace(0.0, 2.0, case["nw"])


MAX_STEPS = 20000          # room of a batch's traces


def prepare(case, seed):
    dev = torch.device("cuda")
    if case["kind"] == "spectrum":
        dip, cur, om = (torch.from_numpy(np.ascontiguousarray(a)).to(dev)
                        for a in _trace(case, seed))
        return dict(kind="spectrum", dt=case["dt"], dip=dip, cur=cur, om=om)
    prec = ks.KS_MIXED if case["mixed"] else ks.KS_FP64
    if case["kind"] == "batch":
        jobs = []
        for i, c in enumerate(_requests(case)):
            d = _describe(c, seed * 100 + i)
            g = ks.Grid(_spec(d), precision=prec)
            serving.set_serving_launch(g, g.spec)
            psi = _states(d, seed * 100 + i, dev)
            jobs.append(ks.Job(g, psi, _vion(d, dev), c["dt"], MAX_STEPS))
        return dict(kind="batch", batch=ks.Batch(jobs), jobs=jobs)
    d = _describe(case, seed)
    vion, psi = _vion(d, dev), _states(d, seed, dev)
    g = ks.Grid(_spec(d), precision=prec)
    s = dict(kind=case["kind"], case=dict(case), grid=g, vion=vion, psi=psi,
             finite=case["per"] == "000",
             t=T_LASER if case["laser"] else 0.0)
    g.update_vlocal(vion, g.density(psi))
    if case["kind"] == "apply":
        s["out"] = torch.empty_like(psi)
    if case["autotune"]:
        g.autotune(psi)
    return s


def run(s):
    kind = s["kind"]
    if kind == "spectrum":
        S = ks.strength_function(s["dip"], s["dt"], 0.01, 0.1, s["om"])
        sig = ks.conductivity(s["cur"], s["dt"], 0.05, 0.1, s["om"])
        return {"strength": S, "sigma": sig}
    if kind == "batch":
        s["batch"].step(1)
        return {"psi": [j.psi for j in s["jobs"]],
                "dipole": [j.dipole for j in s["jobs"]],
                "norms": [j.norms for j in s["jobs"]]}
    g, psi, c = s["grid"], s["psi"], s["case"]
    if kind == "apply":
        for k in range(c["nk"]):
            g.apply_h(psi[k], s["out"][k], k=k, t=s["t"])
        return s["out"]
    if kind in ("etrs", "cfm4"):
        prop = g.propagate_etrs if kind == "etrs" else g.propagate_cfm4
        dip, nrm = prop(psi, s["vion"], c["nsteps"], c["dt"], s["t"],
                        dipole=s["finite"])
        return {"psi": psi, "dipole": dip, "norms": nrm}
    rho = g.density(psi)
    out = {"rho": rho, "norms": g.norms(psi), "gram": g.gram(psi),
           "current": g.current(psi, s["t"]),
           "energy": g.energy(psi, s["vion"], s["t"])}
    if s["finite"]:
        out["dipole"] = g.dipole(rho)
    if c["hartree"]:
        out["hartree"] = g.hartree(rho)
    return out


def work(case):
    """Least bytes and operations of a pass.  H couples every point with the
    projectors of all atoms and the states exceed the caches, so each H.psi
    reads its input states and writes its output once (8 H.psi per step)."""
    kind = case["kind"]
    if kind == "spectrum":
        nt, nw = case["nt"], case["nw"]
        return {"bytes": 8.0 * (2 * nt + 4 * nw), "flops": 2.0 * nt * nw * 8}
    if kind == "batch":
        parts = [work(dict(c, mixed=case["mixed"])) for c in _requests(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    N = case["nx"] * case["ny"] * case["nz"]
    S = case["nk"] * case["ns"]
    rc = 2.5 if case["lmax"] == 2 else 2.0
    sphere = case["natoms"] * 4.19 * rc ** 3 / case["h"] ** 3
    proj = 8.0 * (case["lmax"] + 1) ** 2 * sphere * S
    star = (85.0 + (54.0 if case["laser"] else 0.0)) * N * S
    if kind == "apply":
        return {"bytes": 32.0 * N * S, "flops": star + proj}
    if kind == "observe":
        gram = 8.0 * N * S * case["ns"] / 2
        return {"bytes": 16.0 * N * S, "flops": 2 * (star + proj) + gram}
    b = 32.0 * 8 if not case["mixed"] else 2 * (24.0 + 16 + 16 + 24)
    return {"bytes": b * N * S * case["nsteps"],
            "flops": 8 * (star + proj) * case["nsteps"]}


# ---------------------------------------------------------------------------
# the same results by torch in 64 bits
# ---------------------------------------------------------------------------
class _Plain:
    """H, density, potentials and observables of one system, written out
    with slices, rolls and index lists."""

    def __init__(self, d, vion, dev):
        self.d, self.vion, self.dev = d, vion, dev
        self.n, self.h, self.per = d["n"], d["h"], d["per"]
        self.shape = (self.n[2], self.n[1], self.n[0])
        self.h3 = self.h[0] * self.h[1] * self.h[2]
        self.atoms = [self._sphere(a) for a in range(len(d["Z"]))]
        self.w = torch.from_numpy(np.outer(d["kw"], d["occ"])).to(dev)
        if d["hartree"]:
            self._kernel()

    def _sphere(self, a):
        d, n, h = self.d, self.n, self.h
        lo, i3, w3, r3 = [], [], [], []
        for ax in range(3):
            X, o = d["pos"][a][ax], _axis(n[ax], h[ax], self.per[ax])[0]
            i = np.arange(int(np.floor((X - d["rc"] - o) / h[ax])) - 1,
                          int(np.ceil((X + d["rc"] - o) / h[ax])) + 2)
            if not self.per[ax]:
                i = i[(i >= 0) & (i < n[ax])]
            w = i // n[ax]
            i3.append(i - w * n[ax])
            w3.append(w)
            r3.append(_axis(n[ax], h[ax], self.per[ax])[i3[ax]]
                      + w * n[ax] * h[ax] - X)
        z, y, x = np.meshgrid(r3[2], r3[1], r3[0], indexing="ij")
        r2 = x * x + y * y + z * z
        m = r2 < d["rc"] * d["rc"]
        iz, iy, ix = np.meshgrid(i3[2], i3[1], i3[0], indexing="ij")
        idx = ((iz * n[1] + iy) * n[0] + ix)[m]
        wz, wy, wx = np.meshgrid(w3[2], w3[1], w3[0], indexing="ij")
        T = np.stack([wx[m] * n[0] * h[0], wy[m] * n[1] * h[1],
                      wz[m] * n[2] * h[2]])
        x, y, z, r2 = x[m], y[m], z[m], r2[m]
        rad = (np.exp(-r2 / (2 * d["sigma"] ** 2))
               * (1 - r2 / d["rc"] ** 2) ** 2)
        p = np.stack([np.ones_like(x), x, y, z, x * y, y * z, z * x,
                      x * x - y * y, 3 * z * z - r2])[:(d["lmax"] + 1) ** 2]
        p = p * rad
        p /= np.sqrt((p * p).sum(1, keepdims=True) * self.h3)
        l = np.array([0, 1, 1, 1, 2, 2, 2, 2, 2])[:len(p)]
        t = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to(self.dev)
        return (t(idx), t(p), t(T), t(d["E"][a][l].astype(complex)),
                t(np.stack([x, y, z])))

    def _bloch(self, k, at):
        idx, p, T, E, r = at
        kp = torch.from_numpy(self.d["kpts"][k]).to(self.dev)
        return p * torch.exp(1j * (kp[:, None] * T).sum(0))

    def shift(self, f, ax, m, k):
        """f at the point m steps along axis ax (0 or wrapped outside)."""
        dim = f.dim() - 1 - ax
        n = self.n[ax]
        g = torch.roll(f, -m, dim)
        edge = g.narrow(dim, n - m, m) if m > 0 else g.narrow(dim, 0, -m)
        if self.per[ax]:
            ang = self.d["kpts"][k][ax] * n * self.h[ax]
            edge *= complex(math.cos(ang), math.sin(math.copysign(1, m) * ang))
        else:
            edge.zero_()
        return g

    def laser(self, t):
        A0, om, T = self.d["laser"][:3]
        a = 0.0
        if A0 != 0.0 and 0 <= t <= T:
            a = A0 * math.sin(math.pi * t / T) ** 2 * math.cos(om * t)
        return [a * p for p in self.d["laser"][3:]]

    def apply(self, psi, k, v, A, a2):
        """H psi for [ns, N], in groups of states."""
        out = torch.empty_like(psi)
        grp = max(1, (1 << 25) // psi.shape[1])
        P = [self._bloch(k, at) for at in self.atoms]
        for s in range(0, psi.shape[0], grp):
            f = psi[s:s + grp].reshape((-1,) + self.shape)
            o = f * (v.reshape(self.shape) + a2
                     - 0.5 * C_LAP[0] * sum(1 / q ** 2 for q in self.h))
            for ax in range(3):
                for m in range(1, 5):
                    up, dn = self.shift(f, ax, m, k), self.shift(f, ax, -m, k)
                    if A[ax]:
                        o -= (1j * A[ax] * C_GRAD[m] / self.h[ax]) * (up - dn)
                    o -= (0.5 * C_LAP[m] / self.h[ax] ** 2) * up.add_(dn)
            o = o.reshape(f.shape[0], -1)
            f = f.reshape(f.shape[0], -1)
            for at, p in zip(self.atoms, P):
                c = (f[:, at[0]] @ p.T) * (self.h3 * at[3])
                o[:, at[0]] += c @ p.conj()
            out[s:s + grp] = o
        return out

    def density(self, psi):
        rho = torch.zeros(psi.shape[-1], dtype=torch.float64, device=self.dev)
        for k in range(psi.shape[0]):
            for s in range(psi.shape[1]):
                f = torch.view_as_real(psi[k, s])
                rho += self.w[k, s] * (f * f).sum(-1)
        return rho

    def _kernel(self):
        n, h = self.n, self.h
        if self.per[0]:
            g = [2 * np.pi * np.fft.fftfreq(n[a], d=h[a]) for a in range(3)]
            G2 = (g[2][:, None, None] ** 2 + g[1][None, :, None] ** 2
                  + g[0][None, None, :] ** 2)
            K = np.where(G2 > 0, 4 * np.pi / np.where(G2 > 0, G2, 1), 0)
            self.M = self.shape
        else:
            o = [np.fft.fftfreq(2 * n[a], d=1 / (2 * n[a])) * h[a]
                 for a in range(3)]
            r = np.sqrt(o[2][:, None, None] ** 2 + o[1][None, :, None] ** 2
                        + o[0][None, None, :] ** 2)
            # mean of 1/r over a cell of equal sides (closed form)
            cell = (3 * math.log((math.sqrt(3) + 1) / math.sqrt(2))
                    - math.pi / 4) * 2 / h[0]
            r[0, 0, 0] = 1.0
            K = 1 / r
            K[0, 0, 0] = cell
            K = np.fft.fftn(K).real * self.h3
            self.M = tuple(2 * v for v in self.shape)
        self.K = torch.from_numpy(K).to(self.dev)

    def hartree(self, rho):
        f = torch.fft.fftn(rho.reshape(self.shape), s=self.M)
        v = torch.fft.ifftn(f * self.K).real
        return v[:self.n[2], :self.n[1], :self.n[0]].reshape(-1)

    def vx(self, rho):
        return -((3 / math.pi) * rho) ** (1 / 3)

    def potential(self, rho):
        v = self.vion + self.vx(rho)
        return v + self.hartree(rho) if self.d["hartree"] else v

    def dipole(self, rho):
        f = rho.reshape(self.shape)
        X = [torch.from_numpy(_axis(self.n[a], self.h[a], 0)).to(self.dev)
             for a in range(3)]
        return self.h3 * torch.stack([(f.sum((0, 1)) * X[0]).sum(),
                                      (f.sum((0, 2)) * X[1]).sum(),
                                      (f.sum((1, 2)) * X[2]).sum()])

    def norms(self, psi):
        f = torch.view_as_real(psi.reshape(-1, psi.shape[-1]))
        return self.h3 * torch.stack([(q * q).sum() for q in f])

    def exponential(self, psi, v, A, a2, tau, pred):
        """Taylor-4 of exp(-i tau H) psi, and n of the doubled step."""
        out = torch.empty_like(psi)
        rho = torch.zeros(psi.shape[-1], dtype=torch.float64, device=self.dev)
        grp = max(1, (1 << 26) // psi.shape[-1])
        for k in range(psi.shape[0]):
            for s in range(0, psi.shape[1], grp):
                f = psi[k, s:s + grp]
                t, o, p = f, f.clone(), f.clone() if pred else None
                for j in range(1, 5):
                    t = self.apply(t, k, v, A, a2).mul_(-1j * tau / j)
                    o += t
                    if pred:
                        p += (2 ** j) * t
                out[k, s:s + grp] = o
                if pred:
                    q = torch.view_as_real(p)
                    rho += ((q * q).sum(-1)
                            * self.w[k, s:s + grp, None]).sum(0)
        return out, rho

    def etrs(self, psi, nsteps, dt, t0, dipole):
        rho = self.density(psi)
        v, dip, nrm = self.potential(rho), [], [self.norms(psi)]
        if dipole:
            dip.append(self.dipole(rho))
        for i in range(nsteps):
            At, An = self.laser(t0 + i * dt), self.laser(t0 + (i + 1) * dt)
            half, rho = self.exponential(psi, v, At,
                                         0.5 * sum(a * a for a in At),
                                         dt / 2, True)
            psi, _ = self.exponential(half, self.potential(rho), An,
                                      0.5 * sum(a * a for a in An), dt / 2,
                                      False)
            rho = self.density(psi)
            v = self.potential(rho)
            nrm.append(self.norms(psi))
            if dipole:
                dip.append(self.dipole(rho))
        return (psi, torch.stack(dip) if dipole else None, torch.stack(nrm))

    def cfm4(self, psi, nsteps, dt, t0, dipole):
        q = math.sqrt(3)
        rho = self.density(psi)
        past, dip, nrm = [self.potential(rho)], [], [self.norms(psi)]
        if dipole:
            dip.append(self.dipole(rho))
        for i in range(nsteps):
            c = (0.5 - q / 6, 0.5 + q / 6)
            A = [np.array(self.laser(t0 + (i + x) * dt)) for x in c]
            h = len(past)
            V = [sum(past[j] * float(np.prod([(x + m) / (m - j)
                                              for m in range(h) if m != j]))
                     for j in range(h)) for x in c]
            for w in ((3 + 2 * q) / 6, (3 - 2 * q) / 6):
                psi, _ = self.exponential(
                    psi, w * V[0] + (1 - w) * V[1],
                    list(w * A[0] + (1 - w) * A[1]),
                    0.5 * float(w * A[0] @ A[0] + (1 - w) * A[1] @ A[1]),
                    dt / 2, False)
            rho = self.density(psi)
            past = [self.potential(rho)] + past[:3]
            nrm.append(self.norms(psi))
            if dipole:
                dip.append(self.dipole(rho))
        return (psi, torch.stack(dip) if dipole else None, torch.stack(nrm))

    def current(self, psi, t):
        A = self.laser(t)
        J = np.zeros(3)
        for k in range(psi.shape[0]):
            f = psi[k].reshape((-1,) + self.shape)
            w = self.w[k]
            for ax in range(3):
                o = torch.zeros_like(f)
                for m in range(1, 5):
                    up, dn = self.shift(f, ax, m, k), self.shift(f, ax, -m, k)
                    o -= (0.5 * m * C_LAP[m] / self.h[ax]) * (up - dn)
                    o -= (1j * A[ax] * m * C_GRAD[m]) * (up + dn)
                im = (f.conj() * o).imag.reshape(f.shape[0], -1).sum(1)
                J[ax] += float((w * im).sum()) * self.h3
            f = psi[k]
            for at in self.atoms:
                p, g = self._bloch(k, at), f[:, at[0]]
                c = (g @ p.T) * self.h3
                for ax in range(3):
                    dd = (g * at[4][ax]) @ p.T
                    im = (at[3] * c.conj() * dd).imag.sum(1)
                    J[ax] += 2 * self.h3 * float((w * im).sum())
        return J / np.prod([a * b for a, b in zip(self.n, self.h)])

    def energy(self, psi, t):
        A = self.laser(t)
        a2 = 0.5 * sum(a * a for a in A)
        e = 0.0
        for k in range(psi.shape[0]):
            hp = self.apply(psi[k], k, self.vion, A, a2)
            e += float(((psi[k].conj() * hp).real.sum(1) * self.w[k]).sum())
        rho = self.density(psi)
        e -= 0.75 * (3 / math.pi) ** (1 / 3) * float((rho ** (4 / 3)).sum())
        if self.d["hartree"]:
            e += 0.5 * float((rho * self.hartree(rho)).sum())
        return e * self.h3


def exact(case, seed):
    dev = _device()
    kind = case["kind"]
    if kind == "spectrum":
        dip, cur, om = (torch.from_numpy(a).to(dev)
                        for a in _trace(case, seed))
        n = torch.arange(case["nt"], dtype=torch.float64, device=dev)
        t = n * case["dt"]
        w = torch.ones_like(t)
        w[0] = w[-1] = 0.5
        w = w * torch.exp(-0.1 * t) * case["dt"]
        ph = om[:, None] * t
        f = w * (dip[:, 2] - dip[0, 2])
        S = 2 * om / (math.pi * 0.01) * (torch.sin(ph) * f).sum(1)
        g = w * cur[:, 0]
        return {"strength": S,
                "sigma": torch.complex((torch.cos(ph) * g).sum(1),
                                       -(torch.sin(ph) * g).sum(1)) / 0.05}
    if kind == "batch":
        out = {"psi": [], "dipole": [], "norms": []}
        for i, c in enumerate(_requests(case)):
            d = _describe(c, seed * 100 + i)
            p = _Plain(d, _vion(d, dev), dev)
            psi, dip, nrm = p.etrs(_states(d, seed * 100 + i, dev), 1,
                                   c["dt"], 0.0, True)
            out["psi"].append(psi)
            for name, v in (("dipole", dip), ("norms", nrm)):
                full = torch.zeros(MAX_STEPS + 1, v.shape[1],
                                   dtype=torch.float64, device=dev)
                full[:len(v)] = v
                out[name].append(full)
        return out
    d = _describe(case, seed)
    p = _Plain(d, _vion(d, dev), dev)
    psi = _states(d, seed, dev)
    t = T_LASER if case["laser"] else 0.0
    finite = case["per"] == "000"
    if kind == "apply":
        v = p.potential(p.density(psi))
        A = p.laser(t)
        return torch.stack([p.apply(psi[k], k, v, A,
                                    0.5 * sum(a * a for a in A))
                            for k in range(case["nk"])])
    if kind in ("etrs", "cfm4"):
        psi, dip, nrm = getattr(p, kind)(psi, case["nsteps"], case["dt"], t,
                                         finite)
        return {"psi": psi, "dipole": dip, "norms": nrm}
    rho = p.density(psi)
    out = {"rho": rho, "norms": p.norms(psi),
           "gram": torch.stack([(q.conj() @ q.T) * p.h3 for q in psi]),
           "current": p.current(psi, t), "energy": p.energy(psi, t)}
    if finite:
        out["dipole"] = p.dipole(rho)
    if case["hartree"]:
        out["hartree"] = p.hartree(rho)
    return out
