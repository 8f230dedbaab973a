"""The work users have this library do, as timed cases: Metropolis sweeps of single
lattices from the smallest to the HBM-streaming size, in FP32 and FP16 storage, at
sizes that fit the tiles and sizes that do not; batched temperature scans and
parallel tempering; the four-replica texel; and hybrid Monte Carlo in its three
forms.  Every case goes through the public classes of the package on their default
schedules, with the record buffers a program keeps between calls.

A case is a dict of plain values:
  kind     lattice, batch, tempering, quad, hmc, batch_hmc or quad_hmc
  L        side of the lattice (single lattices and quads)
  n, every sweeps per pass and the record interval (0: no records)
  n, sizes, scan   lattices of a batch, the sides they are drawn from (comma
           separated) and the seed of that draw (workloads.temperature_scan)
  n_md, eps, traj  leap-frog steps, step size and trajectories per pass
  therm    Metropolis sweeps from the hot start that the program has behind it
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_0811_2111_amd import workloads, xy

SCAN_SIZES = "64,128,256,512,1024"
QUAD_BETAS = workloads.QUAD_4096["betas"]


def listed():
    return [
        # the parity configuration in short calls, a record after every sweep: an
        # interactive run or a test, where a call's latency is all there is
        dict(name="lattice_L32", kind="lattice", L=32, prec="fp32", beta=1.0, delta=1.0, n=10, every=1, therm=0),
        # a side from the middle of the paper's Table 1 (128 .. 2048), a chain with a
        # record every 10 sweeps: too small to fill the device
        dict(name="lattice_L256", kind="lattice", L=256, prec="fp32", beta=1.12, delta=1.0, n=100, every=10, therm=0),
        # a side that no tile divides (finite-size scaling takes whatever sides it needs)
        dict(name="lattice_L1000", kind="lattice", L=1000, prec="fp32", beta=1.0, delta=1.0, n=20, every=10, therm=0),
        # the benchmark's single lattice: state and ping-pong copy inside the last-level cache
        dict(name="lattice_L4096", kind="lattice", L=4096, prec="fp32", beta=1.12, delta=1.0, n=20, every=10, therm=0),
        # the storage study's lattice with binary16 angles
        dict(name="lattice_L8192_fp16", kind="lattice", L=8192, prec="fp16", beta=1.0, delta=1.0, n=10, every=10,
             therm=0),
        # the benchmark's headline: 1 GiB of angles, every observable after every sweep
        dict(name="lattice_L16384", kind="lattice", L=16384, prec="fp32", beta=1.0, delta=1.2, n=10, every=1, therm=0),
        # the 96-lattice temperature scan, sides 64 .. 1024
        dict(name="scan_96", kind="batch", n=96, sizes=SCAN_SIZES, scan=1, sweeps=50, every=10, therm=0),
        # parallel tempering over that scan: rounds of ten sweeps and an exchange
        dict(name="tempering_96", kind="tempering", n=96, sizes=SCAN_SIZES, scan=1, rounds=5, sweeps=10, therm=0),
        # four temperatures side by side in one float4 texel
        dict(name="quad_L4096", kind="quad", L=4096, n=10, every=10, therm=0),
        # the paper's own update on the benchmark's single lattice
        dict(name="hmc_L4096", kind="hmc", L=4096, beta=1.0, traj=2, n_md=20, eps=0.02, therm=20),
        # one trajectory after another of every lattice of the scan
        dict(name="hmc_scan_96", kind="batch_hmc", n=96, sizes=SCAN_SIZES, scan=1, traj=2, n_md=20, eps=0.04,
             therm=20),
        # four replicas integrated together, at the side of the documentation's example
        dict(name="quad_hmc_L1024", kind="quad_hmc", L=1024, traj=5, n_md=20, eps=0.04, therm=20),
    ]


# A drawn case costs at most this many site updates (the largest listed pass: 2.7e9).
MOST_UPDATES = 2.0e9


def _side(rng: random.Random, lo: int, hi: int, step: int) -> int:
    """A side spread over the logarithm of [lo, hi]; half of them a multiple of 64."""
    L = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5 and L >= 64:
        step = 64
    return max(lo, min(hi, step * int(round(L / step))))


def draw(rng: random.Random):
    kind = rng.choice(["lattice"] * 5 + ["batch", "tempering", "quad", "hmc", "batch_hmc", "quad_hmc"])
    beta = round(rng.uniform(0.8, 1.3), 4)
    eps_of = lambda L: 0.04 if L <= 1024 else 0.02  # noqa: E731
    if kind == "lattice":
        L = _side(rng, 16, 12288, 2)
        n = rng.choice([1, 10, 25, 100, 300])
        while n > 1 and n * L * L > MOST_UPDATES:
            n = max(1, n // 5)
        every = rng.choice([e for e in (0, 1, 5, 10) if e <= n])
        return dict(kind=kind, L=L, prec=rng.choice(["fp32", "fp32", "fp32", "fp16"]), beta=beta,
                    delta=round(rng.uniform(0.5, 2.0), 3), n=n, every=every, therm=0)
    if kind in ("batch", "tempering", "batch_hmc"):
        n = int(round(math.exp(rng.uniform(math.log(4), math.log(192)))))
        sizes = rng.choice([SCAN_SIZES, SCAN_SIZES, "32,64,128", "100,200,400", "512"])
        scan = rng.randrange(1, 1000)
        if kind == "batch":
            return dict(kind=kind, n=n, sizes=sizes, scan=scan, sweeps=rng.choice([1, 10, 50]),
                        every=rng.choice([0, 1, 10]), therm=0)
        if kind == "tempering":
            return dict(kind=kind, n=n, sizes=sizes, scan=scan, rounds=rng.choice([1, 5]),
                        sweeps=rng.choice([1, 5, 10]), therm=0)
        return dict(kind=kind, n=n, sizes=sizes, scan=scan, traj=rng.choice([1, 2]), n_md=rng.choice([10, 20]),
                    eps=0.04, therm=20)
    if kind == "quad":
        L = _side(rng, 32, 4096, 32)
        n = rng.choice([1, 10, 25])
        while n > 1 and 4 * n * L * L > MOST_UPDATES:
            n = max(1, n // 5)
        return dict(kind=kind, L=L, n=n, every=rng.choice([e for e in (0, 1, 10) if e <= n]), therm=0)
    if kind == "hmc":
        L = _side(rng, 16, 8192, 2)
        return dict(kind=kind, L=L, beta=beta, traj=rng.choice([1, 2]), n_md=rng.choice([10, 20]), eps=eps_of(L),
                    therm=20)
    L = _side(rng, 32, 4096, 32)
    return dict(kind=kind, L=L, traj=rng.choice([1, 2]), n_md=rng.choice([10, 20]), eps=eps_of(L), therm=20)


def _scan(case):
    w = workloads.temperature_scan(n=case["n"], sizes=[int(s) for s in case["sizes"].split(",")], seed=case["scan"])
    return w["Ls"], w["betas"], w["deltas"]


def _seeds(seed: int, n: int):
    """Philox seeds of n lattices: 64-bit, other ones for another seed."""
    r = random.Random(int(seed))
    return [r.getrandbits(63) for _ in range(n)]


def _views(out):
    """The integer and the floating-point columns of a record buffer, as views."""
    if out is None:
        return {}
    if out.shape[-1] == 9:                                  # HMC: traj, accepted, dH and the sums
        return {"counts": out.view(torch.int64)[..., :2], "sums": out[..., 2:]}
    return {"counts": out.view(torch.int64)[..., :2], "sums": out[..., 2:]}


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    kind, dev = case["kind"], "cuda"
    empty = lambda *shape: torch.empty(shape, dtype=torch.float64, device=dev)  # noqa: E731
    if kind in ("lattice", "hmc"):
        s.h = xy.Lattice(case["L"], seed=_seeds(seed, 1)[0], beta=case["beta"], delta=case.get("delta", 1.0),
                         precision=case.get("prec", "fp32"), device=dev)
        nrec = case["n"] // case["every"] if case.get("every") else 0
        s.out = empty(case["traj"], 9) if kind == "hmc" else empty(nrec, 8) if nrec else None
    elif kind in ("quad", "quad_hmc"):
        s.h = xy.Quad(case["L"], seeds=_seeds(seed, 4), betas=QUAD_BETAS, device=dev)
        nrec = case["n"] // case["every"] if case.get("every") else 0
        s.out = empty(case["traj"], 4, 9) if kind == "quad_hmc" else empty(nrec, 4, 8) if nrec else None
    else:
        Ls, betas, deltas = _scan(case)
        n = len(Ls)
        s.h = xy.Batch(Ls, seeds=_seeds(seed, n), betas=betas, deltas=deltas, device=dev)
        if kind == "batch":
            nrec = case["sweeps"] // case["every"] if case["every"] else 0
            s.out = empty(n, nrec, 8) if nrec else None
        elif kind == "tempering":
            s.out = empty(case["rounds"], n, 8)
            s.rungs = torch.empty((case["rounds"], n), dtype=torch.int32, device=dev)
        else:
            s.out = empty(n, case["traj"], 9)
    if case["therm"]:
        s.h.sweep(case["therm"])
    s.outputs = {"state": s.h.state, **_views(s.out)}
    if kind == "tempering":
        s.outputs["rungs"] = s.rungs
    return s


def run(s):
    c, kind = s.case, s.case["kind"]
    if kind in ("lattice", "quad"):
        s.h.sweep(c["n"], c["every"], out=s.out)
    elif kind == "batch":
        s.h.sweep(c["sweeps"], c["every"], out=s.out)
    elif kind == "tempering":
        s.h.tempering(c["rounds"], c["sweeps"], 1, out=s.out, rungs=s.rungs)
    else:
        s.h.hmc(c["traj"], c["n_md"], c["eps"], out=s.out)
    return s.outputs


# Operations of one site update: half a Philox call (20 multiplications and 40 xors
# for two sites), the proposal, its sine and cosine and the site's, the neighbour
# sums, the energy change and the decision.
OPS_UPDATE = 55
# and of one leap-frog step at one site: sine, cosine, neighbour sums, force, kick, drift.
OPS_STEP = 16


def work(case):
    kind = case["kind"]
    if kind in ("lattice", "hmc"):
        sites, lat = case["L"] ** 2, 1
    elif kind in ("quad", "quad_hmc"):
        sites, lat = 4 * case["L"] ** 2, 4
    else:
        Ls = _scan(case)[0]
        sites, lat = sum(L * L for L in Ls), len(Ls)
    elem = 2 if case.get("prec") == "fp16" else 4
    if kind in ("hmc", "quad_hmc", "batch_hmc"):
        return {"bytes": 2.0 * elem * sites + 72.0 * lat * case["traj"],
                "flops": float(sites) * case["traj"] * (case["n_md"] * OPS_STEP + OPS_UPDATE)}
    if kind == "tempering":
        sweeps, nrec = case["rounds"] * case["sweeps"], case["rounds"]
    else:
        sweeps = case["sweeps"] if kind == "batch" else case["n"]
        nrec = sweeps // case["every"] if case["every"] else 0
    return {"bytes": 2.0 * elem * sites + 64.0 * lat * nrec, "flops": float(sites) * sweeps * OPS_UPDATE}


# ------------------------------------------------------------------ 64-bit values
# The same trajectories in plain torch, from the model's definition: energies,
# decisions, sums and the leap-frog in FP64; the random numbers are exact, and the
# Metropolis proposals carry the roundings that the storage format defines.

_M0, _M1, _W0, _W1, _LOW = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85, 0xFFFFFFFF
_DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    for r in range(10):
        if r:
            k0, k1 = (k0 + _W0) & _LOW, (k1 + _W1) & _LOW
        p0, p1 = c0 * _M0, c2 * _M1                          # 64-bit products, modulo 2^64
        c0, c1, c2, c3 = ((p1 >> 32) & _LOW) ^ c1 ^ k0, p1 & _LOW, ((p0 >> 32) & _LOW) ^ c3 ^ k1, p0 & _LOW
    return c0, c1, c2, c3


def _u01(w):
    return ((w >> 9).double() * 2.0 + 1.0) * 2.0 ** -24


def _words(keys, L, counter, colour, purpose, which):
    """Word 0 (or both) that every site of a colour draws, as uniforms (n, L, L/2)."""
    k0, k1 = keys
    P = (L // 2 + 1) // 2
    idx = (torch.arange(L, device=_DEV)[:, None] * P + torch.arange(P, device=_DEV)[None, :])[None]
    full = lambda v: torch.full_like(idx, v)  # noqa: E731
    x = _philox(full(counter), full(colour), full(purpose), idx, k0, k1)
    pair = lambda a, b: torch.stack([a, b], -1).reshape(a.shape[0], L, 2 * P)[..., :L // 2]  # noqa: E731
    return [_u01(pair(x[q], x[q + 2])) for q in which]


def _neighbours(phi, c):
    """left, right, up, down of the entries of colour c: phi is (n, 2, L, L/2)."""
    oth = phi[:, 1 - c]
    L = oth.shape[1]
    odd = ((torch.arange(L, device=phi.device) + c) & 1).bool()[None, :, None]
    left = torch.where(odd, oth, torch.roll(oth, 1, -1))
    right = torch.where(odd, torch.roll(oth, -1, -1), oth)
    return left, right, torch.roll(oth, 1, -2), torch.roll(oth, -1, -2)


_TURN = 2.0 * math.pi


class _Group:
    """Lattices of one side, advanced together."""

    def __init__(self, L, seeds, betas, deltas, prec="fp32"):
        self.L, self.prec = L, prec
        col = lambda v: torch.tensor(v, device=_DEV)[:, None, None]  # noqa: E731
        self.keys = col([s & _LOW for s in seeds]), col([s >> 32 for s in seeds])
        self.set_params(betas, deltas)
        self.phi = torch.stack([_words(self.keys, L, 0, c, 1, (0,))[0] for c in (0, 1)], 1)
        if prec == "fp16":
            self.phi = self.phi.half().double()

    def set_params(self, betas, deltas):
        self.betas, self.deltas = list(betas), list(deltas)
        self.beta = torch.tensor(self.betas, dtype=torch.float64, device=_DEV)[:, None, None]
        self.width = (torch.tensor(self.deltas, dtype=torch.float64, device=_DEV) / _TURN).float()[:, None, None]

    def sweep(self, counter):
        acc = 0
        for c in (0, 1):
            u1, u2 = _words(self.keys, self.L, counter, c, 0, (0, 1))
            own = self.phi[:, c]
            t = own.float() + self.width * (2.0 * u1 - 1.0).float()
            new = (t.double() - torch.floor(t.double())).float().clamp(max=1.0 - 2.0 ** -24)
            new = (new.half() if self.prec == "fp16" else new).double()
            dE = 0.0
            for nb in _neighbours(self.phi, c):
                dE = dE + torch.cos(_TURN * (own - nb)) - torch.cos(_TURN * (new - nb))
            yes = u2 < torch.exp(-self.beta * dE)
            self.phi[:, c] = torch.where(yes, new, own)
            acc = acc + yes.sum((1, 2))
        return acc

    def sums(self):
        """(n, 6): cx, cy, ix, iy, mx, my."""
        v = [0.0] * 6
        for c in (0, 1):
            own = self.phi[:, c]
            _, right, _, down = _neighbours(self.phi, c)
            a, b = _TURN * (own - right), _TURN * (own - down)
            for q, x in enumerate((torch.cos(a), torch.cos(b), torch.sin(a), torch.sin(b), torch.cos(_TURN * own),
                                   torch.sin(_TURN * own))):
                v[q] = v[q] + x.sum((1, 2))
        return torch.stack(v, -1)

    def trajectory(self, counter, n_md, eps):
        p, old = [], self.phi.clone()
        for c in (0, 1):
            u1, u2 = _words(self.keys, self.L, counter, c, 2, (0, 1))
            p.append(torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(_TURN * u2))
        p = torch.stack(p, 1)

        def force():
            f = [sum(torch.sin(_TURN * (nb - self.phi[:, c])) for nb in _neighbours(self.phi, c)) for c in (0, 1)]
            return self.beta[:, None] * torch.stack(f, 1)

        def energy(s):
            return 0.5 * p.square().sum((1, 2, 3)) - self.beta[:, 0, 0] * (s[:, 0] + s[:, 1])

        before = self.sums()
        h0 = energy(before)
        p = p + 0.5 * eps * force()
        for k in range(n_md):
            t = self.phi + eps * p / _TURN
            self.phi = t - torch.floor(t)
            p = p + (eps if k + 1 < n_md else 0.5 * eps) * force()
        after = self.sums()
        dH = energy(after) - h0
        k0, k1 = (k[:, 0, 0] for k in self.keys)
        z = torch.zeros_like(k0)
        yes = _u01(_philox(z + counter, z, z + 3, z, k0, k1)[0]) < torch.exp(-dH)
        self.phi = torch.where(yes[:, None, None, None], self.phi, old)
        return yes, torch.cat([dH[:, None], torch.where(yes[:, None], after, before)], -1)


def _exact_tempering(case, groups, where, n):
    """Rounds of sweeps and exchanges; `groups` in the order of the sides."""
    ladders = []
    for g in groups:
        rung = sorted(range(len(g.betas)), key=lambda i: (g.betas[i], i))
        ladders.append((rung, [g.betas[i] for i in rung], [g.deltas[i] for i in rung]))
    sums = np.zeros((case["rounds"], n, 6))
    counts = np.zeros((case["rounds"], n, 2), dtype=np.int64)
    rungs = np.zeros((case["rounds"], n), dtype=np.int32)
    K, zero = case["sweeps"], torch.zeros((1,), dtype=torch.int64, device=_DEV)
    for r in range(case["rounds"]):
        for gi, g in enumerate(groups):
            rung, betas, deltas = ladders[gi]
            for k in range(K):
                acc = g.sweep(r * K + k)
            rec = g.sums().cpu().numpy()
            sums[r, where[gi]] = rec
            counts[r, where[gi], 0], counts[r, where[gi], 1] = (r + 1) * K, acc.cpu().numpy()
            for t, i in enumerate(rung):
                rungs[r, where[gi][i]] = t
            E = -(rec[:, 0] + rec[:, 1])
            for t in range(r & 1, len(rung) - 1, 2):
                a, b = rung[t], rung[t + 1]
                u = float(_u01(_philox(zero + r, zero + gi, zero + 4, zero + t, zero + 1, zero)[0]))
                if u < math.exp(min(0.0, (betas[t] - betas[t + 1]) * (E[a] - E[b]))):
                    rung[t], rung[t + 1] = b, a
            where_rung = {i: t for t, i in enumerate(rung)}
            g.set_params([betas[where_rung[i]] for i in range(len(rung))],
                         [deltas[where_rung[i]] for i in range(len(rung))])
    return sums, counts, rungs


def exact(case, seed):
    kind = case["kind"]
    many = kind in ("batch", "tempering", "batch_hmc")
    if many:
        Ls, betas, deltas = _scan(case)
        seeds = _seeds(seed, len(Ls))
        where = [[i for i, v in enumerate(Ls) if v == L] for L in sorted(set(Ls))]
        pick = lambda v, w: [v[i] for i in w]  # noqa: E731
        groups = [_Group(Ls[w[0]], pick(seeds, w), pick(betas, w), pick(deltas, w)) for w in where]
    elif kind in ("quad", "quad_hmc"):
        groups, where = [_Group(case["L"], _seeds(seed, 4), QUAD_BETAS, [1.0] * 4)], [[0, 1, 2, 3]]
    else:
        groups = [_Group(case["L"], _seeds(seed, 1), [case["beta"]], [case.get("delta", 1.0)],
                         case.get("prec", "fp32"))]
        where = [[0]]
    n = sum(len(w) for w in where)
    rungs = None
    for g in groups:
        for k in range(case["therm"]):
            g.sweep(k)
    if kind == "tempering":
        sums, counts, rungs = _exact_tempering(case, groups, where, n)
    elif "hmc" in kind:
        sums, counts = np.zeros((n, case["traj"], 7)), np.zeros((n, case["traj"], 2), dtype=np.int64)
        for g, w in zip(groups, where):
            for j in range(case["traj"]):
                yes, rec = g.trajectory(case["therm"] + j, case["n_md"], case["eps"])
                sums[w, j] = rec.cpu().numpy()
                counts[w, j, 0], counts[w, j, 1] = case["therm"] + j + 1, yes.cpu().numpy()
    else:
        sweeps = case["sweeps"] if many else case["n"]
        nrec = sweeps // case["every"] if case["every"] else 0
        sums, counts = np.zeros((n, nrec, 6)), np.zeros((n, nrec, 2), dtype=np.int64)
        for g, w in zip(groups, where):
            for j in range(1, sweeps + 1):
                acc = g.sweep(case["therm"] + j - 1)
                if nrec and j % case["every"] == 0:
                    r = j // case["every"] - 1
                    sums[w, r] = g.sums().cpu().numpy()
                    counts[w, r, 0], counts[w, r, 1] = case["therm"] + j, acc.cpu().numpy()
    if many:
        state = torch.empty((sum(L * L for L in Ls),), dtype=torch.float64, device=_DEV)
        off = np.concatenate([[0], np.cumsum([L * L for L in Ls])])
        for g, w in zip(groups, where):
            for q, i in enumerate(w):
                state[int(off[i]):int(off[i + 1])] = g.phi[q].reshape(-1)
    elif kind in ("quad", "quad_hmc"):
        state = groups[0].phi.permute(1, 2, 3, 0).contiguous()
        sums, counts = sums.transpose(1, 0, 2), counts.transpose(1, 0, 2)
    else:
        state, sums, counts = groups[0].phi[0], sums[0], counts[0]
    out = {"state": state}
    if sums.size:
        out.update(counts=np.ascontiguousarray(counts), sums=np.ascontiguousarray(sums))
    if rungs is not None:
        out["rungs"] = rungs
    return out
