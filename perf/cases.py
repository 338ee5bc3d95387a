"""The work whose speed is measured: passes through the public entry points as a sampling program
calls them.

A Monte Carlo run of this library is a burn-in from static worldlines, a long series of sweeps
on the settled chains, and between sweeps local moves, reconnection swaps, equal-time
measurements and gradients of log Z_path. The cases below cover each of these over the range of
lattices, slices, batch sizes, fields and precisions of the library's own configurations
(`synth`) and of its tests.

Two kinds of state are used, both made from the seed alone:
  start    the initial state of every run: static worldlines, fields N(0,1) or +-1;
  settled  what the chains look like after the burn-in, from the statistics of chains run for
           60 sweeps. Gaussian-field chains: every worldline of both spins on one site per
           slice, which moves by a step about every tenth slice and keeps a few long jumps.
           Ising-field chains: about N/14 occupied sites per spin and slice (at least one), the
           most popular one holding a tenth of the worldlines. The fields are drawn from their
           exact conditionals given those worldlines.
"""
import math

import numpy as np
import torch

import synth
from paper_2510_13866_amd import fhmc
from paper_2510_13866_amd.sampler import Sampler

DEVICE = "cuda:0"


def _case(name, op, L, L_tau, chains, **more):
    c = dict(name=name, op=op, state="settled", precision="fp32", hs="gauss", L=L, L_tau=L_tau,
             chains=chains, filling=0.5, block=0, U=4.0, dtau=0.05, times=1)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one 4 x 4 chain in FP64, all launch latency (small exact studies)
        _case("sweep_4x4_fp64", "sweep", 4, 16, 1, precision="fp64", dtau=0.1),
        # many small Ising chains, the everyday batch
        _case("sweep_16x16_ising", "sweep", 16, 64, 64, hs="ising", dtau=0.0625),
        # the benchmark shape once the chains have settled: most of a run's time
        _case("sweep_32x32", "sweep", 32, 160, 16),
        # the same chains' burn-in: the first sweeps of every run
        _case("start_32x32", "sweep", 32, 160, 16, state="start", times=2),
        # a parameter scan: 256 chains of mixed sizes, temperatures, couplings and fields
        _case("sweep_uneven", "sweep", 0, 0, 256),
        # low temperature (beta = 32) in blocks of 64 slices
        _case("sweep_32x32_blocks64", "sweep", 32, 1024, 4, block=64, dtau=0.03125),
        # the largest lattice
        _case("sweep_64x64", "sweep", 64, 160, 4),
        # reference runs in FP64
        _case("sweep_32x32_fp64", "sweep", 32, 160, 8, precision="fp64"),
        # gradients of log Z_path: at a fresh state in FP32, and along a settled FP64 chain
        # (gradient-informed moves, kinetic energy)
        _case("grad_32x32", "grad", 32, 128, 8, state="start"),
        _case("grad_32x32_fp64", "grad", 32, 128, 8, precision="fp64"),
        # between sweeps: local link moves and reconnection swaps
        _case("moves_32x32", "moves", 32, 160, 16, times=4),
        # equal-time observables
        _case("measure_32x32", "measure", 32, 160, 16, hs="ising"),
    ]


# The most a drawn case costs: the benchmark batch's worldline-slice-sites.
_MOST = 16 * 1024 * 160 * 1024


def _size(c):
    """Worldline-slices times sites of one pass over the batch."""
    N = c["L"] ** 2
    return c["chains"] * 2 * max(1, round(c["filling"] * N)) * c["L_tau"] * N


def draw(rng):
    op = rng.choice(["sweep", "sweep", "sweep", "sweep", "filter", "grad", "grad", "energy",
                     "mala", "moves", "measure"])
    fp64 = rng.random() < 0.35
    hs = rng.choice(["gauss", "gauss", "ising"])
    if op == "measure":
        hs = "ising"  # the clusters of both spins on one site have no spin correlations
    start = op in ("sweep", "filter", "grad", "energy", "mala") and rng.random() < 0.3
    if op in ("grad", "energy", "mala"):
        L = rng.choice([4, 6, 8, 9, 12, 16, 18, 24, 27, 32])
        if hs == "gauss" and not start:
            fp64 = True  # strongly clustered fields leave the range of the FP32 adjoint
        if op == "mala":
            fp64, hs = True, "gauss"  # an exact Metropolis step in FP64 only
    elif hs == "gauss" and not fp64:
        # FP32 plans re-filter clustered blocks in FP64 at these sizes
        L = rng.choice([4, 6, 8, 9, 12, 16, 18, 24, 27, 32, 48, 64])
    else:
        L = rng.choice([4, 6, 8, 9, 12, 16, 18, 24, 27, 32, 36, 48, 64])
    c = _case("", op, L, 0, 0, hs=hs, state="start" if start else "settled",
              precision="fp64" if fp64 else "fp32")
    del c["name"]
    c["L_tau"] = int(round(math.exp(rng.uniform(math.log(12), math.log(400)))))
    c["chains"] = int(round(math.exp(rng.uniform(0, math.log(64)))))
    c["filling"] = rng.choice([0.5, 0.5, round(rng.uniform(0.1, 0.6), 3)])
    c["U"] = round(rng.uniform(2.0, 6.0), 3)
    c["dtau"] = rng.choice([0.03125, 0.05, 0.0625, 0.1])
    if op in ("sweep", "filter") and c["L_tau"] >= 40 and rng.random() < 0.4:
        c["block"] = rng.choice([20, 32, 33, c["L_tau"] // 2 + 1])
    if op == "moves":
        c["times"] = rng.randint(1, 6)
    most = _MOST
    if fp64 and op in ("sweep", "filter"):
        most //= 16 if L > 32 else 2
    if op in ("grad", "energy", "mala"):
        most //= 4
    if L > 32 and not fp64 and op in ("sweep", "filter"):
        most //= 4
    while _size(c) > most and c["chains"] > 1:
        c["chains"] = max(1, c["chains"] * 2 // 3)
    if _size(c) > most:
        c["L_tau"] = max(12, int(c["L_tau"] * most / _size(c)))
        c["block"] = min(c["block"], c["L_tau"])
    return c


# ---- inputs ---------------------------------------------------------------------------------

def _descs(case, seed):
    if case["L"] == 0:
        d = synth.config_uneven(case["chains"])
        return [synth.half_filled(x.L, x.L_tau, x.hs_kind, x.U, x.dtau, seed=seed * 1000 + i)
                for i, x in enumerate(d)]
    n = max(1, round(case["filling"] * case["L"] ** 2))
    kind = synth.HS_GAUSS if case["hs"] == "gauss" else synth.HS_HIRSCH
    return [synth.ChainDesc(L=case["L"], L_tau=case["L_tau"], n_up=n, n_dn=n, hs_kind=kind,
                            block_len=case["block"], t=1.0, U=case["U"], dtau=case["dtau"],
                            seed=seed * 1000 + i) for i in range(case["chains"])]


def _closed_walks(rng, L, L_tau, n, hop, jumps):
    """n site paths [L_tau, n] that close in tau: excursions that go out and come back, `hop` of
    the slices with a unit step, and `jumps` pairs of long jumps per path."""
    step = np.zeros((2, L_tau, n), dtype=np.int64)
    unit = np.array([[1, -1, 0, 0], [0, 0, 1, -1]])
    for k in range(max(1, round(hop * L_tau / 2)) + jumps):
        at = rng.integers(0, L_tau, size=(2, n))
        if k < jumps:
            d = rng.integers(-(L // 3), L // 3 + 1, size=(2, n))
        else:
            d = unit[:, rng.integers(0, 4, size=n)]
        for a in range(2):
            step[a][at[0], np.arange(n)] += d[a]
            step[a][at[1], np.arange(n)] -= d[a]
    xy = [(rng.integers(0, L, size=n) + np.cumsum(step[a], axis=0)) % L for a in range(2)]
    return xy[0] + L * xy[1]


def _potential(d):
    """(coefficient of the field in log W up, down)."""
    if d.hs_kind == synth.HS_GAUSS:
        a = math.sqrt(abs(d.U) * d.dtau)
        return a, a
    lam = math.acosh(math.exp(d.dtau * d.U / 2.0))
    return lam, -lam


def _state(case, d, seed, i):
    """(aux, paths) of one chain as float64 [L_tau, N] and int32 [L_tau, n]."""
    rng = np.random.default_rng([seed, i])
    if case["state"] == "start":
        return synth.initial_aux(d, rng_seed=[seed, i]), synth.initial_paths(d)
    if d.hs_kind == synth.HS_GAUSS:
        paths = np.repeat(_closed_walks(rng, d.L, d.L_tau, 1, 0.08, 2), d.n_particles, axis=1)
    else:
        cols = []
        for n in (d.n_up, d.n_dn):
            k = max(1, round(d.N / 14))
            walks = _closed_walks(rng, d.L, d.L_tau, k, 0.04, 0)
            weight = rng.exponential(size=k)
            cols.append(walks[:, rng.choice(k, size=n, p=weight / weight.sum())])
        paths = np.concatenate(cols, axis=1)
    count = [np.zeros((d.L_tau, d.N)), np.zeros((d.L_tau, d.N))]
    rows = np.arange(d.L_tau)[:, None]
    np.add.at(count[0], (np.broadcast_to(rows, (d.L_tau, d.n_up)), paths[:, :d.n_up]), 1.0)
    np.add.at(count[1], (np.broadcast_to(rows, (d.L_tau, d.n_dn)), paths[:, d.n_up:]), 1.0)
    coef, _ = _potential(d)
    if d.hs_kind == synth.HS_GAUSS:
        aux = coef * (count[0] + count[1] - 0.5) + rng.standard_normal((d.L_tau, d.N))
    else:
        up = 0.5 * (1.0 + np.tanh(coef * (count[0] - count[1])))
        aux = np.where(rng.random((d.L_tau, d.N)) < up, 1.0, -1.0)
    return aux, paths.astype(np.int32)


class _State:
    def __init__(self, case, seed):
        self.case = case
        self.descs = _descs(case, seed)
        fp64 = case["precision"] == "fp64"
        flags = fhmc.FH_FLAG_GRAPH if case["op"] == "sweep" else fhmc.FH_FLAG_NONE
        self.S = Sampler(self.descs, fhmc.FH_FP64 if fp64 else fhmc.FH_FP32_MFMA3, flags, DEVICE)
        both = [_state(case, d, seed, i) for i, d in enumerate(self.descs)]
        self.A = self.S.pack_aux([a for a, _ in both])
        self.P = self.S.pack_paths([p for _, p in both])
        if case["state"] == "start":
            self.A0, self.P0 = self.A.clone(), self.P.clone()
        self.at = 0  # sweep index of the next pass
        if case["op"] == "measure":
            n, sites = len(self.descs), sum(d.N for d in self.descs)
            self.obs = [torch.empty(k, dtype=torch.float64, device=DEVICE)
                        for k in (sites, sites, n, n)]


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    op, S, A, P = s.case["op"], s.S, s.A, s.P
    if op == "sweep":
        n = s.case["times"]
        if s.case["state"] == "start":  # a new run from the initial state
            A.copy_(s.A0)
            P.copy_(s.P0)
            s.at = 0
        S.sweep(A, P, s.at, n)
        s.at += n
        return {"aux": A, "paths": P}
    if op == "filter":
        return {"logZ": S.forward_filter(A, P, 0)}
    if op == "grad":
        logZ, grad_aux, grad_t = S.logz_grad(A, P, 0)
        return {"logZ": logZ, "grad_aux": grad_aux, "grad_t": grad_t}
    if op == "energy":
        return {"energy": S.kinetic_energy(A, P, s.descs[0].L_tau // 2)}
    if op == "mala":
        accepted = S.mala_field(A, P, 0, 0.01, s.at)
        s.at += 1
        return {"accepted": accepted, "aux": A}
    if op == "moves":
        S.local_update(A, P, s.at, s.case["times"])
        S.permutation_update(P, s.at, 2)
        s.at += 1
        return {"paths": P}
    fhmc.fh_measure(S.plan, P, *s.obs)
    return {k: v for k, v in zip(("Sk", "Cr", "D", "S2"), s.obs)}


def work(case):
    """What a pass cannot do without: its inputs and outputs once, and its floating work: one
    filter recursion (C f C, 4 L^3 per slice) per distinct start site of each spin and block,
    a 7 x 7 window per draw."""
    size = 8.0 if case["precision"] == "fp64" else 4.0
    op, total = case["op"], {"bytes": 0.0, "flops": 0.0}
    for d in _descs(case, 0):
        sites, lines = float(d.L_tau * d.N), float(d.L_tau * d.n_particles)
        if case["state"] == "start":
            distinct = min(d.n_up, d.N) + min(d.n_dn, d.N)
        elif d.hs_kind == synth.HS_GAUSS:
            distinct = 2
        else:
            distinct = min(d.n_particles, 2 * max(1, round(d.N / 14)))
        filters = 4.0 * d.L ** 3 * d.L_tau * distinct
        if op == "sweep":
            total["bytes"] += 2 * sites * size + 2 * lines * 4
            total["flops"] += filters + 98.0 * lines
        elif op == "filter":
            total["bytes"] += sites * size + d.n_particles * (4 + 8)
            total["flops"] += filters
        elif op in ("grad", "energy", "mala"):
            evaluations = 2 if op == "mala" else 1
            total["bytes"] += (1 if op == "energy" else 2) * sites * size + d.n_particles * 4
            total["flops"] += evaluations * 2 * filters
        elif op == "moves":
            total["bytes"] += sites * size + 2 * lines * 4
            total["flops"] += 20.0 * lines * case["times"]
        else:
            total["bytes"] += lines * 4 + 2 * d.N * 8
            total["flops"] += 2 * 5.0 * sites * math.log2(d.N) / 2
    times = case["times"] if op == "sweep" else 1
    return {k: v * times for k, v in total.items()}


# ---- the same results in 64 bits, from their definitions --------------------------------------

def _bessel(n, z):
    return math.fsum(math.exp((2 * k + n) * math.log(z / 2) - math.lgamma(k + 1) -
                              math.lgamma(k + n + 1)) for k in range(30))


def _hop(L, t, dtau):
    """Circulant C[x, y] = g(x - y) of one dimension and its t-derivative (device, float64);
    g(d) = sum of the Bessel functions I_n(2 t dtau) over n = d mod L."""
    z = 2.0 * t * dtau
    value = {n: _bessel(n, z) for n in range(0, 4 * L + 42)}
    g, dg = np.zeros(L), np.zeros(L)
    for n in range(-(4 * L + 40), 4 * L + 41):
        g[n % L] += value[abs(n)]
        dg[n % L] += dtau * (value[abs(n - 1)] + value[abs(n + 1)])
    at = (np.arange(L)[:, None] - np.arange(L)[None, :]) % L
    return [torch.from_numpy(v[at]).to(DEVICE) for v in (g, dg)]


def _conv(C, D, f):
    """Sum over r' of C(y - y') D(x - x') f(x', y') for rows f [n, L, L] (y, x)."""
    return torch.matmul(torch.matmul(C, f), D)


def _block_forward(C, W, shift, logw0, start, length, sites):
    """Normalised filter rows and log Z before the end weight of blocks from `sites`."""
    L_tau, L = W.shape[0], C.shape[0]
    f = torch.zeros(len(sites), L * L, dtype=torch.float64, device=DEVICE)
    f[torch.arange(len(sites), device=DEVICE), sites] = 1.0
    f = f.view(-1, L, L)
    log = logw0[start].view(-1)[sites].clone()
    rows = [f]
    for j in range(1, length):
        l = (start + j) % L_tau
        f = _conv(C, C, f) * W[l]
        total = f.sum((1, 2))
        f = f / total[:, None, None]
        log += torch.log(total) + shift[l]
        rows.append(f)
    return rows, log


def _weights(case, d, aux, spin):
    """(W~, log shift, log W) [L_tau, L, L] of one spin, from the field as the plan holds it."""
    a = torch.from_numpy(aux).to(DEVICE)
    if case["precision"] == "fp32":
        a = a.float().double()
    log = (_potential(d)[spin] * a).view(d.L_tau, d.L, d.L)
    shift = log.amax((1, 2))
    return torch.exp(log - shift[:, None, None]), shift, log


def _exact_filter(case, seed):
    out = []
    for i, d in enumerate(_descs(case, seed)):
        aux, paths = _state(case, d, seed, i)
        C, _ = _hop(d.L, d.t, d.dtau)
        B = d.block_len or d.L_tau
        blocks = -(-d.L_tau // B)
        for spin, (lo, hi) in enumerate(((0, d.n_up), (d.n_up, d.n_particles))):
            W, shift, log = _weights(case, d, aux, spin)
            z = torch.zeros(hi - lo, dtype=torch.float64, device=DEVICE)
            for b in range(blocks):
                length = B if b < blocks - 1 else d.L_tau - (blocks - 1) * B
                first = b * B
                ends = np.stack([paths[first, lo:hi], paths[(first + length) % d.L_tau, lo:hi]])
                pairs, which = np.unique(ends, axis=1, return_inverse=True)
                a, e = (torch.from_numpy(v.astype(np.int64)).to(DEVICE) for v in pairs)
                rows, lz = _block_forward(C, W, shift, log, first, length, a)
                end = _conv(C, C, rows[-1]).view(len(a), -1)
                lz = lz + torch.log(end[torch.arange(len(a), device=DEVICE), e])
                z += lz[torch.from_numpy(which.reshape(-1)).to(DEVICE)]
            out.append(z)
    return {"logZ": torch.cat(out)}


def _exact_grad(case, seed, anchor):
    """log Z_path, d/d aux and d/dt per chain: forward rows, backward messages, marginals."""
    descs = _descs(case, seed)
    logZ, grad_t, grad_aux = [], [], []
    for i, d in enumerate(descs):
        aux, paths = _state(case, d, seed, i)
        C, D = _hop(d.L, d.t, d.dtau)
        ga = torch.zeros(d.L_tau, d.L, d.L, dtype=torch.float64, device=DEVICE)
        z = dt = 0.0
        for spin, (lo, hi) in enumerate(((0, d.n_up), (d.n_up, d.n_particles))):
            coef = _potential(d)[spin]
            W, shift, log = _weights(case, d, aux, spin)
            sites, count = np.unique(paths[anchor, lo:hi], return_counts=True)
            for at in range(0, len(sites), 512):
                a = torch.from_numpy(sites[at:at + 512].astype(np.int64)).to(DEVICE)
                n = torch.from_numpy(count[at:at + 512].astype(np.float64)).to(DEVICE)
                rows, lz = _block_forward(C, W, shift, log, anchor, d.L_tau, a)
                u = rows[0]  # the ring closes on the anchor site
                end = _conv(C, C, rows[-1]).view(len(a), -1)
                lz = lz + torch.log(end[torch.arange(len(a), device=DEVICE), a])
                z += float((n * lz).sum())
                for j in range(d.L_tau - 1, -1, -1):
                    l = (anchor + j) % d.L_tau
                    message = _conv(C, C, u)
                    p = rows[j] * message
                    norm = p.sum((1, 2))
                    hop = (rows[j] * (_conv(D, C, u) + _conv(C, D, u))).sum((1, 2))
                    dt += float((n * hop / norm).sum())
                    ga[l] += coef * ((n / norm)[:, None, None] * p).sum(0)
                    u = message * W[l]
                    u = u / u.sum((1, 2))[:, None, None]
                del rows
        logZ.append(z)
        grad_t.append(dt)
        grad_aux.append(ga.reshape(-1))
    as_t = lambda v: torch.tensor(v, dtype=torch.float64)  # noqa: E731
    if case["op"] == "energy":
        return {"energy": as_t([-d.t / (d.L_tau * d.dtau) * g for d, g in zip(descs, grad_t)])}
    return {"logZ": as_t(logZ), "grad_aux": torch.cat(grad_aux), "grad_t": as_t(grad_t)}


def _exact_measure(case, seed):
    out = {"Sk": [], "Cr": [], "D": [], "S2": []}
    for i, d in enumerate(_descs(case, seed)):
        _, paths = _state(case, d, seed, i)
        p = torch.from_numpy(paths.astype(np.int64)).to(DEVICE)
        up, dn = (torch.zeros(d.L_tau, d.N, dtype=torch.float64, device=DEVICE).scatter_add_(
            1, q, torch.ones_like(q, dtype=torch.float64)) for q in (p[:, :d.n_up], p[:, d.n_up:]))
        sz = ((up - dn) / 2).view(d.L_tau, d.L, d.L)
        power = torch.fft.fft2(sz).abs() ** 2
        out["Sk"].append((power / d.N).mean(0).reshape(-1))
        out["Cr"].append((torch.fft.ifft2(power).real / d.N).mean(0).reshape(-1))
        out["D"].append((up * dn).mean())
        out["S2"].append(0.75 * ((up - dn) ** 2).mean())
    return {k: torch.cat(v) if k in ("Sk", "Cr") else torch.stack(v) for k, v in out.items()}


def exact(case, seed):
    """None where the outputs are sampled sites and the fields drawn around them."""
    if case["op"] == "measure":
        return _exact_measure(case, seed)
    if case["op"] == "filter" and _size(case) <= _MOST and case["L"] <= 32:
        return _exact_filter(case, seed)
    if case["op"] == "grad":
        return _exact_grad(case, seed, 0)
    if case["op"] == "energy":
        return _exact_grad(case, seed, case["L_tau"] // 2)
    return None
