"""The work that users of this library have it do, as cases to time and compare.

A case is a plain dict; `prepare` makes what a program holds before the call
(the handle with its system set, positions, dL/dF, output buffers), `run` makes
one pass through the public entry points (`irbe.Handle`, `irbe.IRBEForce`,
`dynamics.Langevin`) and returns every output, `work` the bytes and operations
one pass cannot do without, and `exact` the same outputs in plain FP64 torch,
written from the definitions in `include/irbe.h`.

Keys of a case:
  system     "water" (`size` molecules, rigid, 33.4 per nm^3) or "ions" (`size`
             ions, the 1:1 primitive-model electrolyte at density 0.01)
  precision  "mixed" or "fp64"
  call       "forces": build_lists + compute_forces, every step's work;
             "energy": the same with energies and virial;
             "backward": build_lists + compute_forces + compute_forces_backward;
             "autograd": build_lists, then IRBEForce and its gradients;
             "md": build_lists + compute_forces + one Langevin step;
             "skin": one build_lists, then `reuse` force evaluations at moved
             positions (lists kept over several steps)
  lists      "split" (core + sampled shell list), "full" (every pair),
             "stencil" (the batch drawn from the stencil's cells)
  p_shell, p_kspace, r_core: the method's parameters; reuse: see "skin"
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2204_13595_amd import dynamics, inputs, irbe

SEED = 13595
SKIN = {"water": 0.05, "ions": 0.5}
R_SHELL = {"water": 1.2, "ions": 15.0}
LJ_CUT = {"water": 0.0, "ions": 2.0 ** (1.0 / 6.0)}
DT_PS = 0.001


def _case(system, size, call, lists="split", precision="mixed", p_shell=100, p_kspace=100, r_core=0.5, reuse=0):
    return {"system": system, "size": size, "call": call, "lists": lists, "precision": precision,
            "p_shell": p_shell, "p_kspace": p_kspace, "r_core": r_core, "reuse": reuse}


def listed():
    return [
        # the smallest systems of the tests and the smoke check: launch latency; energies in FP64 over every pair
        dict(_case("water", 512, "energy", lists="full", precision="fp64"), name="water512_full_energy_fp64"),
        # a step of the NVT water runs (901 molecules, r_core 0.7 nm, p = 200): the MD loop at its usual size
        dict(_case("water", 901, "md", p_kspace=200, r_core=0.7), name="water901_md_step"),
        # force matching: forces and their gradients through autograd (water4k)
        dict(_case("water", 4096, "autograd"), name="water4k_force_matching"),
        # the constant-energy box (98,304 atoms, p = 200), lists rebuilt every step
        dict(_case("water", 32768, "forces", p_kspace=200), name="water32k_forces"),
        # a training step in double precision on the same box
        dict(_case("water", 32768, "backward", precision="fp64"), name="water32k_backward_fp64"),
        # lists kept over ten steps with a skin, a box that is no power of two
        dict(_case("water", 100003, "skin", reuse=10), name="water100003_skin10"),
        # stencil sampling, forward and backward (786,432 atoms)
        dict(_case("water", 262144, "backward", lists="stencil"), name="water262k_stencil_backward"),
        # the 3,145,728-atom box of the benchmark: forces, forces with the backward, and the full-list comparison
        dict(_case("water", 1048576, "forces"), name="water1M_forces"),
        dict(_case("water", 1048576, "backward"), name="water1M_backward"),
        dict(_case("water", 1048576, "forces", lists="full"), name="water1M_full_forces"),
        # the electrolyte of the scaling runs at 10^6 ions: lists every step, and kept over 20 steps with a skin
        dict(_case("ions", 1000000, "forces", p_shell=10, r_core=5.0), name="ions1M_forces"),
        dict(_case("ions", 1000000, "skin", p_shell=10, r_core=5.0, reuse=20), name="ions1M_skin20"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.25:
        call = rng.choice(["forces", "energy", "backward", "skin"])
        lists = "split" if call == "backward" else rng.choice(["split", "split", "full"])
        return _case("ions", 2 * _log_int(rng, 2560, 500000), call, lists=lists, p_shell=rng.choice([5, 10, 20]),
                     p_kspace=rng.choice([50, 100, 200]), r_core=rng.choice([4.5, 5.0, 6.0]),
                     reuse=rng.choice([5, 10, 20]) if call == "skin" else 0)
    call = rng.choice(["forces", "forces", "energy", "backward", "backward", "autograd", "md", "skin"])
    precision = rng.choice(["mixed", "mixed", "mixed", "fp64"])
    lists = "split" if call in ("md", "autograd") else rng.choice(["split", "split", "split", "full", "stencil"])
    hi = 16384 if call in ("md", "autograd") else 65536 if precision == "fp64" else 600000
    if lists == "full" and call == "backward":
        hi = min(hi, 65536)
    if call == "skin":
        hi = min(hi, 200000)
    return _case("water", _log_int(rng, 560, hi), call, lists=lists, precision=precision,
                 p_shell=rng.choice([37, 50, 100, 100, 150, 200]), p_kspace=rng.choice([50, 100, 200, 333]),
                 r_core=rng.choice([0.5, 0.5, 0.6, 0.7]), reuse=rng.choice([3, 10]) if call == "skin" else 0)


def _box(case):
    return (case["size"] / 33.45) ** (1.0 / 3.0) if case["system"] == "water" else (case["size"] / 0.01) ** (1.0 / 3.0)


def _system(case, seed):
    """The seeded system, its start positions, the moved ones (equal unless lists
    are kept) and dL/dF, in the case's precision."""
    if case["system"] == "water":
        w = inputs.make_water(case["size"], _box(case), seed=seed)
    else:
        w = inputs.electrolyte(1, seed=seed, box=_box(case), n_anions=case["size"] // 2)
    dev = torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")
    dt = torch.float64 if case["precision"] == "fp64" else torch.float32
    gen = torch.Generator(device="cpu").manual_seed(seed)
    pos = torch.tensor(w.pos, device=dev, dtype=dt)
    moved, grad = pos, None
    if case["call"] == "skin":
        # displacements of just under half the skin: the largest the kept lists allow
        reach = SKIN[case["system"]] / (2.0 * math.sqrt(3.0)) * 0.99
        moved = pos + ((2.0 * torch.rand(pos.shape, generator=gen, dtype=dt) - 1.0) * reach).to(dev)
    if case["call"] in ("backward", "autograd"):
        grad = torch.randn(pos.shape, generator=gen, dtype=dt).to(dev)
    return w, pos, moved, grad


def _method(case):
    """Handle parameters besides the box and precision."""
    ions = case["system"] == "ions"
    return dict(beta=math.sqrt(0.03) if ions else 3.0, r_core=case["r_core"], r_shell=R_SHELL[case["system"]],
                p_shell=0 if case["lists"] == "full" else case["p_shell"], p_kspace=case["p_kspace"], seed=SEED,
                coulomb_k=1.0 if ions else 138.935458, lj_cut=LJ_CUT[case["system"]],
                skin=SKIN[case["system"]] if case["call"] == "skin" else 0.0)


def _step_of(seed):
    return 1 + seed % 1000003


def prepare(case, seed):
    w, pos, moved, grad = _system(case, seed)
    dev, dt = pos.device, pos.dtype
    h = irbe.Handle(w.n_atoms, w.box, precision=case["precision"], device=dev,
                    shell_source="stencil" if case["lists"] == "stencil" else "list", **_method(case))
    q = torch.tensor(w.charge, dtype=dt, device=dev)
    h.set_system(torch.tensor(w.atom_type, device=dev), q, torch.tensor(w.molecule, device=dev), w.lj_sigma, w.lj_eps)
    st = {"case": case, "h": h, "pos": pos, "moved": moved, "grad": grad, "step": _step_of(seed)}
    if case["call"] == "autograd":
        st["x"] = pos.clone().requires_grad_(True)
        st["q"] = q.clone().requires_grad_(True)
        st["sigma"] = torch.tensor(w.lj_sigma, dtype=torch.float64, device=dev, requires_grad=True)
        st["eps"] = torch.tensor(w.lj_eps, dtype=torch.float64, device=dev, requires_grad=True)
    elif case["call"] == "md":
        groups, lengths, inv_mass = dynamics.water_topology(case["size"])
        kT = dynamics.KB * 298.0
        st["dyn"] = dynamics.Langevin(inv_mass, groups, lengths, dt=DT_PS, gamma=1.0, kT=kT, seed=seed + 2,
                                      precision=case["precision"], device=dev)
        gen = torch.Generator(device="cpu").manual_seed(seed + 1)
        st["x0"] = pos.double()
        v = torch.randn(pos.shape, generator=gen, dtype=torch.float64) * np.sqrt(kT * inv_mass)[:, None]
        st["v0"] = v.to(dev)
        st["x"], st["v"], st["force"], st["copy"] = st["x0"].clone(), st["v0"].clone(), pos.clone(), pos.clone()
    elif case["call"] == "skin":
        st["out"] = [torch.empty_like(pos) for _ in range(case["reuse"])]
    else:
        st["force"] = torch.empty_like(pos)
    return st


def run(st):
    h, call, step = st["h"], st["case"]["call"], st["step"]
    h.build_lists(st["pos"], step)
    if call == "forces":
        return h.compute_forces(st["pos"], step, out=st["force"])
    if call == "energy":
        return h.compute_forces(st["pos"], step, out=st["force"], energy=True)
    if call == "backward":
        f = h.compute_forces(st["pos"], step, out=st["force"])
        return (f, *h.compute_forces_backward(st["pos"], step, st["grad"]))
    if call == "autograd":
        leaves = [st["x"], st["q"], st["sigma"], st["eps"]]
        f = irbe.IRBEForce.apply(*leaves, h, step)
        return (f.detach(), *torch.autograd.grad(f, leaves, grad_outputs=st["grad"]))
    if call == "skin":
        for k, out in enumerate(st["out"]):
            h.compute_forces(st["moved"], step + k, out=out)
        return st["out"]
    # "md": every pass starts from the same snapshot, so that it can be repeated
    st["x"].copy_(st["x0"])
    st["v"].copy_(st["v0"])
    h.compute_forces(st["pos"], step, out=st["force"])
    st["dyn"].step(st["x"], st["v"], st["force"], step, pos_copy=st["copy"])
    return st["x"], st["v"], st["force"], st["copy"]


def work(case):
    """Bytes: positions, charges, types and molecule ids read once per pass (moved
    positions once per evaluation), outputs written once. Operations: 8 for the
    distance test of each pair within r_shell of the lists, 60 per evaluated pair
    and evaluation (about twice that in a backward), 20 per atom and k-vector in
    the structure factor and in the force."""
    n = case["size"] * (3 if case["system"] == "water" else 1)
    rs = 8 if case["precision"] == "fp64" else 4
    dens = n / _box(case) ** 3
    ball = lambda r: 4.0 / 3.0 * math.pi * r ** 3 * dens
    within, core = min(ball(R_SHELL[case["system"]]), n), min(ball(case["r_core"]), n)
    pairs = within if case["lists"] == "full" else core + min(case["p_shell"], within - core)
    evals = case["reuse"] if case["call"] == "skin" else 1
    nbytes = n * (3 * rs + rs + 8) + n * 3 * rs * evals
    flops = n * within * 8 + n * evals * (60 * pairs + 40 * case["p_kspace"])
    if case["call"] == "skin":
        nbytes += n * 3 * rs * evals
    if case["call"] in ("backward", "autograd"):
        nbytes += n * (6 * rs + rs)
        flops += n * (120 * pairs + 80 * case["p_kspace"])
    if case["call"] == "md":
        nbytes += n * (4 * 24 + 3 * rs)
        flops += n * 200
    return {"bytes": float(nbytes), "flops": float(flops)}


# ---------------------------------------------------------------------------
# The outputs in FP64, from the definitions: fixed-point positions, cells, lists
# in canonical order, Philox samples, pair sums, structure factors.
# ---------------------------------------------------------------------------
M32 = 0xFFFFFFFF
MAX_CANDIDATES = 2.0e9  # beyond this the plain evaluation would take too long


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


class _Words:
    """One word stream per id, each with its own position."""

    def __init__(self, seed, step, ids, tag):
        self.k = (seed & M32, seed >> 32)
        self.ids, self.c2, self.c3 = ids, step & M32, ((step >> 32) << 1) | tag
        self.at = torch.zeros_like(ids)

    def next(self, rows=slice(None)):
        ids, at = self.ids[rows], self.at[rows].clone()
        fixed = torch.zeros_like(ids)
        words = torch.stack(_philox(ids, at // 4, fixed + self.c2, fixed + self.c3, *self.k))
        self.at[rows] = at + 1
        return words.gather(0, (at % 4)[None])[0]

    def below(self, bound):
        """Uniform integers in [0, bound): multiply-shift with rejection."""
        def parts(w, b):
            m = w * b  # below 2^48
            return m >> 32, m & M32
        r, low = parts(self.next(), bound)
        thr = (2 ** 32 - bound) % bound
        bad = torch.nonzero(low < thr)[:, 0]
        while bad.numel():
            r[bad], low[bad] = parts(self.next(bad), bound[bad])
            bad = bad[low[bad] < thr[bad]]
        return r


class _Exact:
    def __init__(self, case, seed):
        self.case = case
        w, pos, moved, grad = _system(case, seed)
        m = _method(case)
        self.w, self.m, self.dev = w, m, pos.device
        self.L = w.box
        self.grad = None if grad is None else grad.double()
        self.q = torch.tensor(w.charge, device=self.dev, dtype=pos.dtype).double()
        self.type = torch.tensor(w.atom_type, device=self.dev).long()
        self.mol = torch.tensor(w.molecule, device=self.dev).long()
        self.sigma = torch.tensor(w.lj_sigma, device=self.dev, dtype=torch.float64)
        self.eps = torch.tensor(w.lj_eps, device=self.dev, dtype=torch.float64)
        self.n, self.step = w.n_atoms, _step_of(seed)
        self.full, self.stencil = case["lists"] == "full", case["lists"] == "stencil"
        rc, rs = m["r_core"] + m["skin"], m["r_shell"] + m["skin"]
        self.n_c = int(math.floor(self.L / rc))
        reach = int(math.floor(rs * float(self.n_c) / self.L)) + 1
        if 2 * reach + 1 <= self.n_c:
            self.lo, self.span = -reach, 2 * reach + 1
        else:
            self.lo, self.span = -((self.n_c - 1) // 2), self.n_c
        self.t_core, self.t_shell = self._thr(m["r_core"]), self._thr(m["r_shell"])
        self.tl_core, self.tl_shell = self._thr(rc), self._thr(rs)
        self.tl_lo = self._thr(max(m["r_core"] - m["skin"], 0.0))
        self.s0, self.s = self._quantize(pos), self._quantize(moved)
        per_cell = self.n / self.n_c ** 3
        self.candidates = self.n * self.span ** 3 * per_cell

    def _thr(self, r):
        t = r * 4294967296.0 / self.L
        return int(math.floor(t * t))

    def _quantize(self, x):
        u = x.double() * (1.0 / self.L)
        return torch.round((u - torch.floor(u)) * 4294967296.0).long() & M32

    def _diff(self, s, i, j):
        d = (s[j] - s[i]) & M32
        return torch.where(d >= 2 ** 31, d - 2 ** 32, d)

    def _within(self, d, thr):
        """D^2 <= thr without overflow (thr < 2^62)."""
        t = math.isqrt(thr)
        ok = (d.abs() <= t).all(1)
        d = torch.where(ok[:, None], d, 0)
        xy = d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]
        ok &= xy <= thr
        return ok & (torch.where(ok, xy, 0) + d[:, 2] * d[:, 2] <= thr)

    def lists(self):
        """Core pairs and, in canonical order, the atoms the batch is drawn from
        (offsets and flat indices, caller ids)."""
        n, n_c, dev = self.n, self.n_c, self.dev
        cell = (self.s0 * n_c) >> 32
        cid = (cell[:, 2] * n_c + cell[:, 1]) * n_c + cell[:, 0]
        order = torch.argsort(self.s0[:, 0], stable=True)
        order = order[torch.argsort(cid[order], stable=True)]
        start = torch.zeros(n_c ** 3 + 1, dtype=torch.long, device=dev)
        start[1:] = torch.cumsum(torch.bincount(cid, minlength=n_c ** 3), 0)
        off = torch.arange(self.lo, self.lo + self.span, device=dev)
        oz, oy = off.repeat_interleave(self.span), off.repeat(self.span)
        core_i, core_j, sh_i, sh_j = [], [], [], []
        per = max(1, int(1.2e7 / max(1.0, self.candidates / n)))
        for a in range(0, n, per):
            i = order[a:a + per]
            c = cell[i]
            row = (((c[:, 2:3] + oz) % n_c) * n_c + (c[:, 1:2] + oy) % n_c) * n_c
            x0 = (c[:, 0:1] + self.lo) % n_c
            la = torch.clamp(n_c - x0, max=self.span)
            seg0 = torch.stack([start[row + x0], start[row]], 2)
            seg1 = torch.stack([start[row + x0 + la], start[row + self.span - la]], 2)
            seg0, length = seg0.flatten(), (seg1 - seg0).flatten()
            base = torch.cumsum(length, 0) - length
            at = torch.arange(int(length.sum()), device=dev) + (seg0 - base).repeat_interleave(length)
            j = order[at]
            ii = i.repeat_interleave(length.reshape(len(i), -1).sum(1))
            d = self._diff(self.s0, ii, j)
            keep = (ii != j) & ~((self.mol[ii] >= 0) & (self.mol[ii] == self.mol[j]))
            shell = keep & self._within(d, self.tl_shell)
            core = shell & self._within(d, self.tl_core)
            if self.full:
                drawn_from = shell
            else:
                drawn_from = shell & ~core if self.m["skin"] == 0 else shell & ~self._within(d, self.tl_lo)
                core_i.append(ii[core].int())
                core_j.append(j[core].int())
            if self.stencil:
                sh_i.append(ii.int())
                sh_j.append(torch.where(drawn_from, j, -1).int())
            else:
                sh_i.append(ii[drawn_from].int())
                sh_j.append(j[drawn_from].int())
        cat = lambda t: torch.cat(t) if t else torch.zeros(0, dtype=torch.int32, device=dev)
        self.core = (cat(core_i), cat(core_j))
        self.shell_i, self.shell_j = cat(sh_i), cat(sh_j)
        self.n_s = torch.bincount(self.shell_i, minlength=n)
        # a flat entry's place in its atom's list
        first = torch.zeros(n, dtype=torch.long, device=dev)
        idx = order
        first[idx] = torch.cumsum(self.n_s[idx], 0) - self.n_s[idx]
        self.rank = torch.arange(len(self.shell_i), device=dev) - first[self.shell_i.long()]

    def batch(self, step):
        """Pairs of the batch and their weights at `step` (every entry of the full list)."""
        if self.full:
            return self.shell_i, self.shell_j, torch.ones(len(self.shell_i), device=self.dev, dtype=torch.float64)
        p = self.m["p_shell"]
        big = torch.nonzero(self.n_s > p)[:, 0]
        most = int(self.n_s.max())
        taken = torch.ones((self.n, most), dtype=torch.bool, device=self.dev)
        taken[big] = False
        words = _Words(SEED, step, big, 0)
        for c in range(p):
            t = self.n_s[big] - p + c
            r = words.below(t + 1)
            v = torch.where(taken[big, r], t, r)
            taken[big, v] = True
        i = self.shell_i.long()
        sel = taken[i, self.rank] & (self.shell_j >= 0)
        weight = torch.where(self.n_s > p, self.n_s.double() / p, 1.0)
        return self.shell_i[sel], self.shell_j[sel], weight[i[sel]]

    def kvectors(self, step):
        a = math.pi / (self.m["beta"] * self.L)
        wt = lambda k: math.exp(-((a * float(k)) ** 2))
        top = 0
        while wt(top + 1) >= 2.0 ** -64:
            top += 1
        axis = [wt(k) for k in range(-top, top + 1)]
        H = 0.0
        for v in axis:
            H += v
        U, c = [], 0.0
        for v in axis:
            c += v
            U.append(min(int((c / H) * 2.0 ** 64), 2 ** 64 - 1))
        U[-1] = 2 ** 64 - 1
        U = np.array(U, dtype=np.uint64)
        P = self.m["p_kspace"]
        words = _Words(SEED, step, torch.arange(P), 1)
        m = np.zeros((P, 3), dtype=np.int64)
        todo = torch.arange(P)
        while todo.numel():
            for ax in range(3):
                hi, lo = words.next(todo).numpy().astype(np.uint64), words.next(todo).numpy().astype(np.uint64)
                u = (hi << np.uint64(32)) | lo
                m[todo.numpy(), ax] = np.minimum(np.searchsorted(U, u, side="right"), 2 * top) - top
            todo = todo[torch.tensor((m[todo.numpy()] == 0).all(1))]
        S = H ** 3 - 1.0
        k = 2.0 * math.pi / self.L * m
        coef = self.m["coulomb_k"] * (S / P) * 4.0 * math.pi / self.L ** 3 / (k ** 2).sum(1)
        to = lambda x: torch.tensor(x, device=self.dev)
        return to(m), to(k), to(coef)

    def pair_terms(self, i, j, u, q, sigma, eps, excluded):
        """d (r_j - r_i), the force factor f = phi d and the energies of pairs."""
        i, j = i.long(), j.long()
        d = self._diff(self.s, i, j).double() * (self.L / 4294967296.0)
        if u is not None:
            d = d + u[j] - u[i]
        r2 = (d * d).sum(1)
        r = torch.sqrt(r2)
        b = self.m["beta"]
        qq = self.m["coulomb_k"] * q[i] * q[j]
        gauss = 2.0 * b / math.sqrt(math.pi) * torch.exp(-b * b * r2)
        if excluded:
            erf = torch.erf(b * r)
            return d, -qq / r2 * (gauss - erf / r), -qq * erf / r, torch.zeros_like(r)
        erfc = torch.erfc(b * r)
        t = self.type[i] * 2 + self.type[j]
        sg, ep = sigma[t], eps[t]
        x6 = (sg * sg / r2) ** 3
        cut = self.m["lj_cut"]
        on = torch.ones_like(r) if cut == 0.0 else (r < cut * sg).double()
        shift = 0.0 if cut == 0.0 else 4.0 * ep * (cut ** -12 - cut ** -6)
        phi = -qq / r2 * (erfc / r + gauss) - on * ep * (48.0 * x6 * x6 - 24.0 * x6) / r2
        return d, phi, qq * erfc / r, on * (4.0 * ep * (x6 * x6 - x6) - shift)

    def groups(self, step):
        """(pairs i, j, weight, excluded) of every short-range sum at `step`, in chunks."""
        bi, bj, bw = self.batch(step)
        if self.m["skin"] > 0.0:
            ok = self._annulus(bi, bj)
            bi, bj, bw = bi[ok], bj[ok], bw[ok]
        ci, cj = self.core
        if self.m["skin"] > 0.0 and len(ci):
            ok = torch.cat([self._within(self._diff(self.s, a.long(), b.long()), self.t_core)
                            for a, b in zip(ci.split(1 << 24), cj.split(1 << 24))])
            ci, cj = ci[ok], cj[ok]
        xi = xj = torch.zeros(0, dtype=torch.int32, device=self.dev)
        if self.case["system"] == "water":
            a = torch.arange(self.n, device=self.dev)
            xi = a.repeat_interleave(2)
            xj = torch.stack([a // 3 * 3 + (a + 1) % 3, a // 3 * 3 + (a + 2) % 3], 1).flatten()
        for i, j, w, ex in ((ci, cj, None, False), (bi, bj, bw, False), (xi, xj, None, True)):
            for at in range(0, len(i), 1 << 22):
                e = at + (1 << 22)
                wt = torch.ones(len(i[at:e]), device=self.dev, dtype=torch.float64) if w is None else w[at:e]
                yield i[at:e], j[at:e], wt, ex

    def _annulus(self, i, j):
        out = []
        for a, b in zip(i.split(1 << 24), j.split(1 << 24)):
            d = self._diff(self.s, a.long(), b.long())
            ok = self._within(d, self.t_shell)
            out.append(ok if self.full else ok & ~self._within(d, self.t_core))
        return torch.cat(out)

    def phases(self, m, lo, hi):
        ph = (self.s @ m[lo:hi].t()) & M32 if self.s.device.type == "cpu" else \
            (self.s[:, None, :] * m[lo:hi][None]).sum(2) & M32
        return torch.where(ph >= 2 ** 31, ph - 2 ** 32, ph).double() * (2.0 * math.pi / 4294967296.0)

    def forward(self, step):
        f_sr = torch.zeros((self.n, 3), device=self.dev, dtype=torch.float64)
        f_ex = torch.zeros_like(f_sr)
        ev = torch.zeros(11, device=self.dev, dtype=torch.float64)
        for i, j, w, ex in self.groups(step):
            d, phi, uc, ul = self.pair_terms(i, j, None, self.q, self.sigma, self.eps, ex)
            (f_ex if ex else f_sr).index_add_(0, i.long(), (w * phi)[:, None] * d)
            ev[4 if ex else 0] += 0.5 * (w * uc).sum()
            ev[1] += 0.5 * (w * ul).sum()
            for c, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                ev[5 + c] -= 0.5 * (w * phi * d[:, a] * d[:, b]).sum()
        f = f_sr + f_ex
        if not self.full:
            f = f - f_sr.mean(0)
        m, k, coef = self.kvectors(step)
        beta = self.m["beta"]
        for lo in range(0, len(m), 16):
            th = self.phases(m, lo, lo + 16)
            c, s = torch.cos(th), torch.sin(th)
            re, im = self.q @ c, self.q @ s
            g = (c * im - s * re) * coef[lo:lo + 16]
            f = f - self.q[:, None] * (g @ k[lo:lo + 16])
            kk, cf = k[lo:lo + 16], coef[lo:lo + 16]
            ul = 0.5 * cf * (re * re + im * im)
            ev[2] += ul.sum()
            geo = 2.0 * (1.0 / (kk * kk).sum(1) + 1.0 / (4.0 * beta * beta))
            for e, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                ev[5 + e] += (ul * ((1.0 if a == b else 0.0) - geo * kk[:, a] * kk[:, b])).sum()
        ev[3] = -self.m["coulomb_k"] * beta / math.sqrt(math.pi) * (self.q * self.q).sum()
        return f, ev

    def backward(self, step):
        """dL/dr, dL/dq, dL/dsigma, dL/deps of L = sum G.F at fixed samples and lists."""
        leaves = [torch.zeros((self.n, 3), device=self.dev, dtype=torch.float64), self.q.clone(), self.sigma.clone(),
                  self.eps.clone()]
        total = [torch.zeros_like(x) for x in leaves]
        for x in leaves:
            x.requires_grad_(True)
        u, q, sigma, eps = leaves

        def add(loss):
            for acc, g in zip(total, torch.autograd.grad(loss, leaves, allow_unused=True)):
                if g is not None:
                    acc += g
        G = self.grad
        Gc = G if self.full else G - G.mean(0)
        for i, j, w, ex in self.groups(step):
            d, phi, _, _ = self.pair_terms(i, j, u, q, sigma, eps, ex)
            add((w * phi * (d * (G if ex else Gc)[i.long()]).sum(1)).sum())
        m, k, coef = self.kvectors(step)
        for lo in range(0, len(m), 8):
            kk = k[lo:lo + 8]
            th = self.phases(m, lo, lo + 8) + u @ kk.t()
            c, s = torch.cos(th), torch.sin(th)
            re, im = q @ c, q @ s
            add(-(q[:, None] * (c * im - s * re) * coef[lo:lo + 8] * (G @ kk.t())).sum())
        return total


def exact(case, seed):
    e = _Exact(case, seed)
    passes = case["reuse"] if case["call"] == "skin" else 1
    pairs = e.n * (e.case["p_shell"] if not e.full else 800)
    if e.candidates > MAX_CANDIDATES or (e.n > 10 ** 6) or pairs * passes > 4e8:
        return None
    e.lists()
    if case["call"] == "skin":
        return [e.forward(e.step + k)[0] for k in range(passes)]
    f, ev = e.forward(e.step)
    if case["call"] == "energy":
        return f, ev
    if case["call"] == "md":
        # (the constrained Langevin step that follows is compared with itself only)
        return None, None, f, None
    if case["call"] in ("backward", "autograd"):
        gp, gq, gs, ge = e.backward(e.step)
        return (f, gp, gq, gs, ge) if case["call"] == "autograd" else (f, gp, gq, torch.cat([gs, ge]))
    return f
