"""Timed cases: the work a user of this framework has it do, through its public entry points.

Families (`kind`):
  increment  one load increment of a single model (`Solver.load_step`): prologue, pseudo-transient sweeps until the
             residual and the FP64 certificate meet the tolerance, epilogue; a cyclic loading schedule
             (`Solver.set_strain_rate`), so that every pass solves an increment of the same size.  Read back: the
             velocities, the pressure and the accumulated plastic strain.
  sweeps     a window of pseudo-transient sweeps of the first yielding increment (`Solver.sweep`): what a large model
             spends its hours on, cut to a length that can be timed.  Read back: the velocities and the pressure.
             The larger 2D models have the regularised return (`vp`): without it the sweep at which each of their many
             equal cells yields is a matter of rounding, and no two programs agree on the fields.
  batch      one load increment of many 2D models of uneven sizes (`Batch.load_step`): a parameter sweep.
  forward, gradient, train
             the warm-start network: inference, one gradient of one sample, and a few optimiser steps over a set of
             samples (`Net.forward`, `Net.gradient`, `Net.train`).

Fields come back from the solver as float64 arrays; where the iteration fields are FP32 (`precision` "fp32") a program
keeps them in that type, and so do the outputs here.

`exact` is plain torch in float64, written from the equations: staggered grid, backward Euler in pseudo-time for
pressure and deviator, radial return of the physical trial at the centres, mean multiplier at the shear points.
"""
import math

import numpy as np
import torch

from ep_workloads import Model
from paper_2305_01701_amd import ep

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # the smallest model in use (63 x 63, FP64, tol 1e-8): one increment is thousands of very short sweeps
        dict(name="increment 2d 63 fp64", kind="increment", nx=63, ny=63, nz=0, precision="fp64", tol=1e-8, freeze=0),
        # the 2:1 domain of the symmetry study in FP64, frozen plasticity after 16 nx iterations
        dict(name="increment 2d 383x191 fp64", kind="increment", nx=383, ny=191, nz=0, precision="fp64", tol=1e-7,
             freeze=16, vp=5e-4),
        # a 2D increment with FP32 iteration fields, the precision hand-over and frozen plasticity
        dict(name="increment 2d 511 fp32", kind="increment", nx=511, ny=511, nz=0, precision="fp32", tol=1e-6,
             freeze=16, vp=5e-4),
        # a small 3D increment with FP32 iteration fields: residual checks every ten short sweeps
        dict(name="increment 3d 63 fp32", kind="increment", nx=63, ny=63, nz=63, precision="fp32", tol=1e-6,
             freeze=0),
        # the 2D production size, FP32 iteration fields
        dict(name="sweeps 2d 1023 fp32", kind="sweeps", nx=1023, ny=1023, nz=0, precision="fp32", n=4000, het=False,
             vp=5e-4),
        # a ragged 2D grid with a per-cell shear modulus in FP64 (the heterogeneous setup's finishing sweeps)
        dict(name="sweeps 2d 777x1010 fp64 het", kind="sweeps", nx=777, ny=1010, nz=0, precision="fp64", n=2000,
             het=True, vp=5e-4),
        # the 3D production size, FP32 iteration fields: the largest case
        dict(name="sweeps 3d 255 fp32", kind="sweeps", nx=255, ny=255, nz=255, precision="fp32", n=1600, het=False),
        # a ragged 3D grid in FP64 (the finishing sweeps of every large increment)
        dict(name="sweeps 3d 190x127x101 fp64", kind="sweeps", nx=190, ny=127, nz=101, precision="fp64", n=600,
             het=False),
        # a parameter sweep over 24 models of 127^2 to 511^2 cells
        dict(name="batch 2d 24 models fp32", kind="batch", models=24, largest=511, precision="fp32", tol=1e-6),
        # warm-start inference on a small grid: launches and latency
        dict(name="forward 31 base 32", kind="forward", nx=31, ny=31, nz=31, base=32),
        # one gradient at the training size (127^3): forward, input gradients and weight gradients of all layers
        dict(name="gradient 127 base 32", kind="gradient", nx=127, ny=127, nz=127, base=32),
        # a few optimiser steps on a ragged mid-size grid with the narrow network
        dict(name="train 70x61x45 base 16", kind="train", nx=70, ny=61, nz=45, base=16, steps=8),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["increment", "increment", "sweeps", "sweeps", "sweeps", "batch", "forward", "gradient", "train"])
    prec = rng.choice(["fp32", "fp64"])
    if kind == "increment":
        if rng.random() < 0.6:
            nx = _spread(rng, 31, 400)
            ny = max(16, int(nx * rng.uniform(0.5, 1.0)))
            return dict(kind=kind, nx=nx, ny=ny, nz=0, precision=prec, tol=rng.choice([1e-6, 1e-7]),
                        freeze=16 if nx > 100 else rng.choice([0, 16]), vp=5e-4 if nx > 100 else 0.0)
        nx = _spread(rng, 16, 70)
        return dict(kind=kind, nx=nx, ny=max(12, int(nx * rng.uniform(0.6, 1.0))),
                    nz=max(12, int(nx * rng.uniform(0.6, 1.0))), precision=prec, tol=1e-6, freeze=0)
    if kind == "sweeps":
        het = rng.random() < 0.3
        if rng.random() < 0.5:
            nx, ny = _spread(rng, 100, 1200), _spread(rng, 100, 1200)
            return dict(kind=kind, nx=nx, ny=ny, nz=0, precision=prec, n=rng.randrange(500, 2000), het=het,
                        vp=5e-4)
        nx, ny, nz = (_spread(rng, 30, 200) for _ in range(3))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=prec, n=rng.randrange(100, 400), het=het)
    if kind == "batch":
        return dict(kind=kind, models=rng.randrange(4, 24), largest=rng.choice([127, 255, 383]), precision=prec, tol=1e-6)
    hi = {"forward": 96, "gradient": 110, "train": 64}[kind]
    nx = _spread(rng, 14, hi)
    ny, nz = (max(10, int(nx * rng.uniform(0.6, 1.0))) for _ in range(2))
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, base=rng.choice([16, 32]))
    if kind == "train":
        c["steps"] = rng.randrange(2, 9)
    return c


# ----------------------------------------------------------------- the inputs


def _gen(seed, k=0):
    return np.random.Generator(np.random.PCG64([int(seed), k]))


def _axis(n, length):
    return -0.5 * length + (np.arange(n) + 0.5) * (length / n)


def _smooth(r, axes, amp):
    """1 + a few long waves of total amplitude amp over the cells (x fastest)."""
    out = 1.0
    for _ in range(3):
        w = amp / 3
        for d, ax in enumerate(axes):                        # axes[0] = x, the last array axis
            k, ph = r.integers(1, 4), r.uniform(0, 2 * math.pi)
            w = w * np.cos(math.pi * k * ax + ph).reshape((-1,) + (1,) * d)
        out = out + w
    return out


def _model(case, seed, k=0):
    """A pure-shear model with a weak inclusion off the centre and a smoothly varying cohesion: its parameters, the
    cohesion and, for a heterogeneous case, the shear modulus of every cell."""
    r = _gen(seed, k)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    d3 = nz > 0
    lx, ly, lz = 1.0, 1.0 if d3 else round(ny / nx, 2) or 0.01, 1.0
    nmax = max(nx, ny, nz)
    m = Model(ndim=3 if d3 else 2, nx=nx, ny=ny, nz=nz if d3 else 1, lx=lx, ly=ly, lz=lz, tol=case.get("tol", 1e-6),
              dt=(1.4e-3 if d3 else 1e-3) * (1.0 if case["kind"] == "increment" else 0.5), freeze_iter=case.get("freeze", 0) * nmax, max_iter=400 * nmax,
              shear=1.2 if case.get("het") else 1.0, eta_vp=case.get("vp", 0.0))
    axes = [_axis(nx, lx), _axis(ny, ly)] + ([_axis(nz, lz)] if d3 else [])
    rad = r.uniform(0.1, 0.15) * min(lx, ly)
    d2 = 0.0
    for d, ax in enumerate(axes):
        d2 = d2 + ((ax - r.uniform(-0.1, 0.1) * min(lx, ly)) ** 2).reshape((-1,) + (1,) * d)
    coh = m.c0 * _smooth(r, axes, 0.1)
    coh = np.ascontiguousarray(np.where(d2 < rad * rad, 0.5 * coh, coh)).ravel()
    shear = None
    if case.get("het"):                                      # softer towards the inclusion, at most the reference
        shear = np.ascontiguousarray((1.2 - 0.2 * np.exp(-d2 / 0.04)) * _smooth(r, axes, 0.05) / 1.06).ravel()
    return m, coh, shear


PREC = {"fp64": ep.EP_FP64, "fp32": ep.EP_FP32_FIELDS}


def _batch_sizes(case):
    """Cells per side of the models: the sizes of the batched workload up to the largest, in a fixed uneven order."""
    r = _gen(case["models"], 1)
    return [int(r.choice([s for s in (127, 255, 383, 511) if s <= case["largest"]])) for _ in range(case["models"])]


def _batch_models(case, seed):
    r = _gen(seed, 1)
    out = []
    for k, n in enumerate(_batch_sizes(case)):
        m, coh, _ = _model(dict(kind="batch", nx=n, ny=n, nz=0, tol=case["tol"]), seed, 100 + k)
        m = m.with_(phi_deg=float(r.uniform(20.0, 40.0)), eta_vp=float(r.uniform(3e-4, 6e-4)))
        out.append((m, coh * float(r.uniform(0.8, 1.4))))
    return out


def _net_channels(base):
    c, c2, c4 = base, 2 * base, 4 * base
    return [(16, c), (c, c), (c, c2), (c2, c2), (c2, c4), (c4, c4), (c4, c2), (c2, c2), (c2, c), (c, c), (c, 16)]


def _net_weights(case, seed):
    """He-normal weights with small biases and a head that is not zero, as after some training: flat float32."""
    g = torch.Generator().manual_seed(int(seed) * 7 + 1)
    flat = []
    for l, (ci, co) in enumerate(_net_channels(case["base"])):
        sd = math.sqrt(2.0 / (27 * ci)) * (0.5 if l == 10 else 1.0)
        flat += [torch.randn(co * 27 * ci, generator=g) * sd, torch.randn(co, generator=g) * 0.02]
    return torch.cat(flat).numpy()


def _net_sample(case, seed, k, dims):
    """Features (11 of 16 channels) and targets on the grid's cells, zero on the padding of the network volume."""
    D, H, W = dims
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 131 + k)
    x = torch.zeros((D, H, W, 16), device="cuda")
    t = torch.zeros((D, H, W, 4), device="cuda")
    s = (slice(0, case["nz"]), slice(0, case["ny"]), slice(0, case["nx"]))
    f = torch.randn((D, H, W, 11), generator=g, device="cuda")
    f[:, :, 1:] += f[:, :, :-1].clone()
    x[s + (slice(0, 11),)] = f[s] * 0.7
    t[s + (slice(0, 3),)] = torch.randn((D, H, W, 3), generator=g, device="cuda")[s] * 0.3
    return x, t


def _dims(case):
    return tuple((case[k] + 3) // 4 * 4 for k in ("nz", "ny", "nx"))


# ------------------------------------------------------------------- a pass


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind in ("increment", "sweeps"):
        m, coh, shear = _model(case, seed)
        s["solver"] = ep.Solver(m, coh, precision=PREC[case["precision"]], shear=shear)
        s["names"] = ["vx", "vy", "vz", "p"] if case["nz"] else ["vx", "vy", "p"]
        if kind == "increment":
            s["names"] = s["names"] + ["eps_p"]
        s["pass"] = 0
    elif kind == "batch":
        ms = _batch_models(case, seed)
        s["batch"] = ep.Batch([m for m, _ in ms], [c for _, c in ms], precision=PREC[case["precision"]])
        s["views"] = [s["batch"].model(i) for i in range(len(ms))]
    else:
        n = case.get("steps", 1) if kind == "train" else 1
        slots = min(n, 4)
        net = ep.Net(case["nx"], case["ny"], case["nz"], base=case["base"], max_samples=slots)
        net.set_params(_net_weights(case, seed))
        for k in range(slots):
            x, t = _net_sample(case, seed, k, net.dims)
            net.set_sample(k, x.cpu().numpy(), t.cpu().numpy())
        s["net"], s["slots"] = net, list(range(slots))
    return s


def _typed(case, a):
    return a.astype(np.float32) if case["precision"] == "fp32" else a


def _rate(k):
    """Loading schedule of the increment cases: half an increment forward, then back and forth over a whole one."""
    return 0.5 if k == 0 else -1.0 if k % 2 else 1.0


def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "increment":
        r = _rate(s["pass"])
        s["pass"] += 1
        s["solver"].set_strain_rate((r, -r, 0.0))
        s["solver"].load_step()
        return {n: _typed(case, s["solver"].get(n)) for n in s["names"]}
    if kind == "sweeps":
        s["solver"].sweep(case["n"])
        return {n: _typed(case, s["solver"].get(n)) for n in s["names"]}
    if kind == "batch":
        s["batch"].load_step()
        return [{n: _typed(case, v.get(n)) for n in ("vx", "vy")} for v in s["views"]]
    if kind == "forward":
        return s["net"].forward(0)
    if kind == "gradient":
        loss, grad = s["net"].gradient(0)
        return {"loss": np.float32(loss), "grad": grad}
    losses = s["net"].train(s["slots"], case["steps"])
    return {"losses": losses, "weights": s["net"].get_params()}


# -------------------------------------------------------------- what it needs


def _cells(nx, ny, nz):
    return float(nx) * ny * (nz or 1)


def work(case):
    kind = case["kind"]
    if kind in ("increment", "sweeps", "batch"):
        # per sweep and cell: 3D 9 fields read and written, 6 increment-start fields and the cohesion read (25
        # accesses, about 150 operations); 2D 6, 4 and 1 (17 accesses, about 90); per-cell G: one more read.  Sweeps of
        # an increment per cell of its longest side, as counted: about 8 with the regularised return, 17 without it
        # in 2D, 20 in 3D
        size = 4 if case["precision"] == "fp32" else 8
        if kind == "batch":
            models = [(n, n, 0, 8 * n) for n in _batch_sizes(case)]
        else:
            per = 20 if case["nz"] else 8 if case.get("vp") else 17
            n = case["n"] if kind == "sweeps" else per * max(case["nx"], case["ny"], case["nz"])
            models = [(case["nx"], case["ny"], case["nz"], n)]
        total = {"bytes": 0.0, "flops": 0.0}
        for nx, ny, nz, n in models:
            acc = (25 if nz else 17) + (1 if case.get("het") else 0)
            total["bytes"] += n * _cells(nx, ny, nz) * acc * size
            total["flops"] += n * _cells(nx, ny, nz) * (150 if nz else 90)
        return total
    d = _dims(case)
    v0 = float(np.prod(d))
    vols = [v0, v0, v0 / 8, v0 / 8, v0 / 64, v0 / 64, v0 / 8, v0 / 8, v0, v0, v0]
    ch = _net_channels(case["base"])
    flops = sum(54.0 * ci * co * v for (ci, co), v in zip(ch, vols))
    acts = sum(2.0 * co * v for (_, co), v in zip(ch, vols))
    wts = sum(4.0 * (27 * ci + 1) * co for ci, co in ch)
    if kind == "forward":
        return {"bytes": v0 * (32 + 64) + wts, "flops": flops}
    one = {"bytes": v0 * (32 + 16) + 2 * acts + 2 * wts, "flops": 3 * flops - 2.0 * 54 * 16 * ch[0][1] * v0 / 2}
    n = case.get("steps", 1)
    return {k: n * v for k, v in one.items()}


# ---------------------------------------------------------- float64 reference


class _PT:
    """The pseudo-transient iteration of one increment from rest, in float64; arrays in (z,) y, x order."""

    def __init__(self, m, coh, shear, rate):
        self.m, self.d3 = m, m.ndim == 3
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        n = [m.nx, m.ny] + ([m.nz] if self.d3 else [])
        ext = [m.lx, m.ly] + ([m.lz] if self.d3 else [])
        self.n, self.nd = n, len(n)
        self.h = [e / k for e, k in zip(ext, n)]
        full = tuple(n[::-1])
        z = lambda *grow: torch.zeros([n[d] + (1 if d in grow else 0) for d in reversed(range(self.nd))],  # noqa: E731
                                      dtype=torch.float64, device=dev)
        self.c = torch.as_tensor(np.asarray(coh), dtype=torch.float64, device=dev).reshape(full)
        self.v = [z(d) for d in range(self.nd)]
        for d in range(self.nd):
            x = -0.5 * ext[d] + torch.arange(n[d] + 1, dtype=torch.float64, device=dev) * self.h[d]
            shape = [1] * self.nd
            shape[self.nd - 1 - d] = n[d] + 1
            # the initial velocities are those of unit rate; the walls move at the increment's
            self.v[d] += ((1.0, -1.0, 0.0)[d] * x).reshape(shape)
            self._ends(self.v[d], d, (1.0, -1.0, 0.0)[d] * rate * 0.5 * ext[d])
        self.p = z()
        self.t = [z(), z()]
        self.pairs = [(0, 1)] + ([(0, 2), (1, 2)] if self.d3 else [])
        self.s = [z(*pr) for pr in self.pairs]
        re, rr, cfl = 3 * math.sqrt(10) * math.pi / 2, m.r, 0.9 / math.sqrt(self.nd)
        eta = 1.0 / (1.0 / (m.shear * m.dt))
        L, h = max(ext), min(self.h)
        self.gdt = re * eta * cfl * h / (L * (rr + 4.0 / 3.0))
        self.kdt = rr * self.gdt
        self.dtrho = cfl * h * L / (re * eta)
        self.eta, self.L = eta, L
        ph = math.radians(m.phi_deg)
        if self.d3:
            self.A, self.B = (6 * f(ph) / (math.sqrt(3) * (3 - math.sin(ph))) for f in (math.sin, math.cos))
        else:
            self.A, self.B = math.sin(ph), math.cos(ph)
        G = m.shear if shear is None else torch.as_tensor(np.asarray(shear), dtype=torch.float64, device=dev).reshape(full)
        self.ig = 1.0 / (G * m.dt) + torch.zeros_like(self.c)
        self.igs = [self._mean(self.ig, pr) for pr in self.pairs]
        self.ref = 2 * m.shear * rate * m.dt / L
        self.frozen = None

    def ax(self, d):
        return self.nd - 1 - d

    def _ends(self, a, d, w):
        a.select(self.ax(d), 0).fill_(-w)
        a.select(self.ax(d), -1).fill_(w)

    def _diff(self, a, d):
        return torch.diff(a, dim=self.ax(d)) / self.h[d]

    def _pair(self, a, d):
        n = a.shape[self.ax(d)]
        return 0.5 * (a.narrow(self.ax(d), 0, n - 1) + a.narrow(self.ax(d), 1, n - 1))

    def _mean(self, a, pr):
        """Centres to the interior shear points, or shear points to the centres, of the plane `pr`."""
        return self._pair(self._pair(a, pr[0]), pr[1])

    def _in(self, a, *ds):
        for d in ds:
            a = a.narrow(self.ax(d), 1, a.shape[self.ax(d)] - 2)
        return a

    def sweep(self, blend, physical=False, hold=False, old=0.0):
        """One iteration (all old stresses zero); physical: without the pseudo-time terms, velocities kept.
        Returns the momentum and the combined residual."""
        m = self.m
        igt, ikt = (0.0, 0.0) if physical else (1 / self.gdt, 1 / self.kdt)
        ikd = 1.0 / (m.bulk * m.dt)
        S = []
        for (a, b), s in zip(self.pairs, self.s):
            e = torch.zeros_like(s)
            self._in(e, a, b).copy_(self._diff(self._in(self.v[a], a), b) + self._diff(self._in(self.v[b], b), a))
            S.append(e)
        g = [self._diff(self.v[d], d) for d in range(self.nd)]
        div = sum(g)
        pn = (self.p * ikt - div) / (ikt + ikd)
        Sn = [2 * (g[d] - div / 3) for d in range(2)]
        Tn = [self.t[d] * igt + Sn[d] for d in range(2)]
        D = igt + self.ig
        sq = lambda q: 0.5 * (q[0] ** 2 + q[1] ** 2 + ((q[0] + q[1]) ** 2 if self.d3 else 0.0))  # noqa: E731
        sh2 = sum(self._mean(e, pr) ** 2 for e, pr in zip(S, self.pairs))
        if self.frozen is None:
            b = self.A * pn + self.B * self.c
            Y, vp = b.clamp(min=0.0), m.eta_vp

            def back(J, D):                                  # tauII of the return: the bound and the overstress
                return Y + vp * torch.where(b < 0, J / (1 + D * vp), (J - D * b) / (1 + D * vp))

            JS = (sq(Sn) + sh2).sqrt()
            lam = JS / back(JS, self.ig) - self.ig
            if not physical and blend != 0.0:
                f = (D + lam) / (self.ig + lam)
                JT = (sq(Tn) + f * f * sh2).sqrt()
                lt = torch.where(JT / D > Y, JT / back(JT, D) - D, torch.zeros_like(D))
                fin = torch.isfinite(lam) & torch.isfinite(lt)
                lam = torch.where(fin, lam + blend * (lt - lam), lam)
            lam = torch.where(JS / self.ig > Y, lam, torch.zeros_like(lam))
            if hold:
                self.frozen = lam
        else:
            lam = self.frozen
        tn = [T / (D + lam) for T in Tn]
        sn = []
        for e, s, pr, ig in zip(S, self.s, self.pairs, self.igs):
            q = torch.zeros_like(s)
            self._in(q, *pr).copy_(self._in(s * igt + e, *pr) / (igt + ig + self._mean(lam, pr)))
            sn.append(q)
        dia = [tn[0] - pn, tn[1] - pn] + ([-(tn[0] + tn[1]) - pn] if self.d3 else [])
        mom, vn = 0.0, []
        for d in range(self.nd):
            r = self._diff(dia[d], d)
            for q, (a, b) in zip(sn, self.pairs):
                if d in (a, b):
                    r = r + self._diff(self._in(q, d), b if d == a else a)
            mom = torch.maximum(r.abs().max(), torch.as_tensor(mom, dtype=torch.float64, device=r.device))
            vn.append((d, r))
        rate = [(pn - self.p).abs().max() * (m.bulk * m.dt / (self.kdt * self.L))]
        rG = self.eta / (self.gdt * self.L)
        rate += [(x - y).abs().max() * rG for x, y in zip(tn + sn, self.t + self.s)]
        if self.d3:
            rate.append((tn[0] + tn[1] - self.t[0] - self.t[1]).abs().max() * rG)
        self.p, self.t, self.s = pn, tn, sn
        if not physical:
            for d, r in vn:
                self._in(self.v[d], d).add_(r, alpha=self.dtrho)
        return mom, torch.stack([mom] + rate).max()

    def plastic(self):
        """Plastic strain of the increment from the physical stresses of the velocities (J2 of the trial over its
        compliance against the bound)."""
        g = [self._diff(self.v[d], d) for d in range(self.nd)]
        div = sum(g)
        Sn = [2 * (g[d] - div / 3) for d in range(2)]
        p = -div * self.m.bulk * self.m.dt
        J = 0.5 * (Sn[0] ** 2 + Sn[1] ** 2 + ((Sn[0] + Sn[1]) ** 2 if self.d3 else 0.0))
        for (a, b), s in zip(self.pairs, self.s):
            e = torch.zeros_like(s)
            self._in(e, a, b).copy_(self._diff(self._in(self.v[a], a), b) + self._diff(self._in(self.v[b], b), a))
            J = J + self._mean(e, (a, b)) ** 2
        tr = J.sqrt() / self.ig
        b, vp = self.A * p + self.B * self.c, self.m.eta_vp
        Y = b.clamp(min=0.0)
        D = self.ig
        back = Y + vp * torch.where(b < 0, tr * D / (1 + D * vp), D * (tr - b) / (1 + D * vp))
        return 0.5 * self.m.dt * torch.where(tr > Y, D * (tr - back), torch.zeros_like(tr))

    def fields(self, names):
        at = {"vx": 0, "vy": 1, "vz": 2}
        return {n: (self.v[at[n]] if n in at else self.p if n == "p" else self.plastic()).reshape(-1).cpu().numpy()
                for n in names}


def _increment(case, m, coh, shear):
    """The increment of the first pass: as the solver's, with a tolerance a thousand times tighter."""
    q = _PT(m, coh, shear, 0.5)
    mom, _ = q.sweep(0.0, physical=True)
    tol = 1e-3 * m.tol * max(float(mom), q.ref)
    check = 10 if q.d3 else 100
    nmax = max(q.n)
    it, hold = 0, False
    while it < m.max_iter:
        blend = m.pt_blend_late if it >= 16 * nmax else m.pt_blend
        for k in range(check):
            _, res = q.sweep(blend, hold=hold and k == 0)
        it += check
        hold = bool(m.freeze_iter) and it >= m.freeze_iter and q.frozen is None
        if float(res) <= tol:
            break
    q.sweep(0.0, physical=True)
    return q


def _net_exact(case, seed):
    """Forward pass, loss and gradient of the network in float64 (27 shifted products per convolution)."""
    D, H, W = _dims(case)
    dev = "cuda"
    ch = _net_channels(case["base"])

    def split(flat):
        out, o = [], 0
        for ci, co in ch:
            n = co * 27 * ci
            out.append((flat[o:o + n].reshape(co, 27, ci), flat[o + n:o + n + co]))
            o += n + co
        return out

    taps = [(a, b, c) for a in range(3) for b in range(3) for c in range(3)]

    def conv(x, w):
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        d, h, wd = x.shape[:3]
        y = 0
        for t, (a, b, c) in enumerate(taps):
            y = y + xp[a:a + d, b:b + h, c:c + wd].reshape(-1, x.shape[3]) @ w[:, t, :].t()
        return y.reshape(d, h, wd, -1)

    def conv_dx(g, w):
        return conv(g, w.flip(1).permute(2, 1, 0))

    def conv_dw(x, g):
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        d, h, wd = x.shape[:3]
        g2 = g.reshape(-1, g.shape[3])
        dw = torch.stack([g2.t() @ xp[a:a + d, b:b + h, c:c + wd].reshape(-1, x.shape[3]) for a, b, c in taps], 1)
        return torch.cat([dw.reshape(-1), g2.sum(0)])

    def pool(x):
        d, h, w, c = x.shape
        return x.reshape(d // 2, 2, h // 2, 2, w // 2, 2, c).mean((1, 3, 5))

    def up(x):
        return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    def fwd(P, x):
        act = {"x": x}
        lay = lambda k, v: (conv(v, P[k][0]) + P[k][1]).clamp(min=0)  # noqa: E731
        act["a0"] = lay(0, x)
        act["s0"] = lay(1, act["a0"])
        act["p0"] = pool(act["s0"])
        act["a1"] = lay(2, act["p0"])
        act["s1"] = lay(3, act["a1"])
        act["p1"] = pool(act["s1"])
        act["a2"] = lay(4, act["p1"])
        act["b2"] = lay(5, act["a2"])
        act["u1"] = up(act["b2"])
        act["r6"] = lay(6, act["u1"])
        act["c1"] = act["r6"] + act["s1"]
        act["d1"] = lay(7, act["c1"])
        act["u0"] = up(act["d1"])
        act["r8"] = lay(8, act["u0"])
        act["c0"] = act["r8"] + act["s0"]
        act["d0"] = lay(9, act["c0"])
        return conv(act["d0"], P[10][0]) + P[10][1], act

    def grad(P, x, t):
        y, a = fwd(P, x)
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        mask = torch.zeros_like(y)
        mask[:nz, :ny, 1:nx, 0] = 1
        mask[:nz, 1:ny, :nx, 1] = 1
        mask[1:nz, :ny, :nx, 2] = 1
        tt = torch.zeros_like(y)
        tt[..., :4] = t
        e = (y - tt) * mask
        gy = 2 * e / mask.sum()
        G = [None] * 11

        def back(k, inp, z):
            G[k] = conv_dw(a[inp], z)
            return conv_dx(z, P[k][0]) if k else None

        unup = lambda g: pool(g) * 8  # noqa: E731
        z = back(10, "d0", gy) * (a["d0"] > 0)
        gc0 = back(9, "c0", z)
        gd1 = unup(back(8, "u0", gc0 * (a["r8"] > 0)))
        gc1 = back(7, "c1", gd1 * (a["d1"] > 0))
        gb2 = unup(back(6, "u1", gc1 * (a["r6"] > 0)))
        z = back(5, "a2", gb2 * (a["b2"] > 0)) * (a["a2"] > 0)
        gs1 = gc1 + up(back(4, "p1", z)) / 8
        z = back(3, "a1", gs1 * (a["s1"] > 0)) * (a["a1"] > 0)
        gs0 = gc0 + up(back(2, "p0", z)) / 8
        z = back(1, "a0", gs0 * (a["s0"] > 0)) * (a["a0"] > 0)
        back(0, "x", z)
        return float((e * e).sum() / mask.sum()), torch.cat(G)

    w = torch.as_tensor(_net_weights(case, seed), device=dev).double()
    sample = lambda k: tuple(q.double() for q in _net_sample(case, seed, k, (D, H, W)))  # noqa: E731
    if case["kind"] == "forward":
        return fwd(split(w), sample(0)[0])[0].cpu().numpy()
    if case["kind"] == "gradient":
        loss, g = grad(split(w), *sample(0))
        return {"loss": loss, "grad": g.cpu().numpy()}
    m, v, losses = torch.zeros_like(w), torch.zeros_like(w), []
    for k in range(case["steps"]):                            # Adam, learning rate 1e-3
        loss, g = grad(split(w), *sample(k % min(case["steps"], 4)))
        losses.append(loss)
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        w = w - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"losses": np.array(losses), "weights": w.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":                                       # thousands of sweeps of every model: minutes
        return None
    if kind in ("forward", "gradient", "train"):
        return _net_exact(case, seed)
    m, coh, shear = _model(case, seed)
    names = ["vx", "vy", "vz", "p"] if case["nz"] else ["vx", "vy", "p"]
    if kind == "increment":
        if case["freeze"] and case["precision"] == "fp32":
            # the multiplier that is held is the iterate's at that sweep: a value of the path, not of the equations
            return None
        return _increment(case, m, coh, shear).fields(names + ["eps_p"])
    q = _PT(m, coh, shear, 1.0)
    for _ in range(case["n"]):
        q.sweep(m.pt_blend)
    return q.fields(names)
