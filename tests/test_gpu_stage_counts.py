"""Staged backward draws in states that are staged by the rule in force, which every case asserts:
the draws of one recursion per worldline, whatever tier decides them, from the plan's rows in both
precisions and from the FP64 re-filter's slots in its phases A and B."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def clustered(d, k, jump, rng):
    """(paths, walk of each): worldlines spread unevenly over k random walks, one of which jumps."""
    walks = synth.random_walk_paths(synth.ChainDesc(**{**d.__dict__, "n_up": k, "n_dn": 0}),
                                    int(rng.integers(1 << 30)))
    walks[d.L_tau // 2:, 0] = (walks[d.L_tau // 2:, 0] + jump + d.L * jump) % d.N
    w = rng.exponential(size=k) + 0.05
    on = rng.choice(k, size=d.n_particles, p=w / w.sum())
    return walks[:, on], on


def reconnections(d, on, rng):
    """A permutation per spin, of the worldlines on one walk among themselves where `on` is given."""
    perm = np.arange(d.n_particles)
    on = np.zeros(d.n_particles, dtype=int) if on is None else on
    for p0, p1 in ((0, d.n_up), (d.n_up, d.n_particles)):
        for k in range(on.max() + 1):
            at = p0 + np.flatnonzero(on[p0:p1] == k)
            perm[at] = rng.permutation(at)
    return perm


# the first chain's rows end on an odd element, so the next chains' start on one in FP32; more start
# sites than the row buffer holds in 16 x 16, 24 x 24 and 32 x 32; whole and ragged workgroups
ODD = synth.ChainDesc(L=9, L_tau=5, n_up=2, n_dn=1, hs_kind=0, block_len=0, t=1.0, U=4.0, dtau=0.05,
                      seed=3)
CASES = [(8, 9, 64, 2, 0, 1), (8, 12, 130, 126, 2, 5), (12, 10, 140, 172, 3, 20),
         (16, 11, 300, 330, 4, 40), (18, 25, 330, 200, 5, 9), (24, 12, 600, 580, 6, 40),
         (32, 21, 900, 700, 7, 30), (48, 7, 400, 260, 0, 3), (64, 6, 300, 200, 0, 2)]


@pytest.mark.parametrize("L,L_tau,n_up,n_dn,block,walks", CASES)
@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_every_case_is_staged_and_draws_the_same_sites(prec, L, L_tau, n_up, n_dn, block, walks):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    rng = np.random.default_rng(L + L_tau)
    descs = [ODD] + [synth.ChainDesc(L=L, L_tau=L_tau, n_up=n_up, n_dn=n_dn, hs_kind=k,
                                     block_len=block, t=1.0, U=4.0, dtau=0.05, seed=90 + k)
                     for k in range(2)]
    print("staged draws", prec, L, L_tau, n_up, n_dn, block, flush=True)
    aux = [synth.initial_aux(d) for d in descs]
    jump = L // 2 if prec == "fp64" else min(L // 2, 6)  # FP32 holds no hop of 16 + 16 sites
    both = [clustered(d, walks, jump, rng) for d in descs[1:]]
    paths = [synth.initial_paths(ODD)] + [p for p, _ in both]
    perms = [np.arange(3)] + [reconnections(d, None if prec == "fp64" else on, rng)
                              for d, (_, on) in zip(descs[1:], both)]
    nb = -(-L_tau // (block or L_tau))
    room = min(64, 32768 // (L * L * (8 if prec == "fp64" else 4)))
    want = {}
    for share, bound in ((0, 1.0), (1, 1.0), (1, 1e7), (1, float("inf"))):
        S = Sampler(descs, precision)
        assert fhmc.lib.fh_debug_share_filters(S.plan, share) == 0
        assert fhmc.lib.fh_debug_inflate_window_bound(S.plan, bound) == 0
        S.set_permutation(perms)
        A = S.pack_aux(aux)
        for s in range(3):
            P = S.pack_paths(paths)
            S.forward_filter(A, P, s)
            counts = fhmc.fh_debug_staged(S.plan)
            assert counts[0] == (4 * nb if share else 0), (s, counts)
            if share and walks > room:
                assert counts[2] > 4 * nb  # several groups of start sites
            S.backward_sample(P, s)
            assert fhmc.fh_debug_rescue(S.plan)[0] == 0  # drawn from the plan's rows, all of them
            if share:
                assert torch.equal(P, want[s]), (s, bound)
            else:
                want[s] = P
        assert S.status() == (0, -1)
        S.close()


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("prec,L,block,n_up,n_dn", [
    ("mfma3", 32, 0, 150, 90), ("mfma3", 16, 4, 60, 41), ("fp32", 48, 0, 200, 150),
    ("mfma3", 48, 5, 200, 150), ("mfma3", 64, 0, 300, 200), ("mfma3", 64, 4, 300, 200)])
def test_refiltered_chains_draw_staged_in_phases_a_and_b(prec, L, block, n_up, n_dn, graph):
    """A field whose weights leave FP32's range in the first sweep: chains queued whole take phase B in
    plans with 48 x 48 or 64 x 64 lattices, one recursion per start site, and the next sweeps' held
    chains phase A. Sites and fields equal those of k_rescue, a recursion per worldline."""
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP32 if prec == "fp32" else fhmc.FH_FP32_MFMA3
    descs = [synth.ChainDesc(L=L, L_tau=11, n_up=n_up, n_dn=n_dn, hs_kind=0, block_len=block, t=1.0,
                             U=4.0, dtau=0.02, seed=70 + k) for k in range(2)]
    print("phases A and B", prec, L, block, graph, flush=True)
    rng = np.random.default_rng(L + block)
    aux = []
    for k, d in enumerate(descs):
        a = rng.standard_normal((d.L_tau, d.N))
        if k == 0:  # the other chain stays in range
            a -= 500.0
            a[:, (d.L // 2) * (d.L + 1)] = 0.0
        aux.append(a)
    # every worldline of a spin on one site a slice, near the origin
    paths = [np.repeat(rng.integers(0, 2, (d.L_tau, 2)) * np.array([1, d.L]), [d.n_up, d.n_dn], axis=1)
             for d in descs]
    got, phases = {}, []
    nb = -(-11 // (block or 11))
    for share in (0, 1):
        S = Sampler(descs, precision, fhmc.FH_FLAG_GRAPH if graph else 0)
        assert fhmc.lib.fh_debug_share_filters(S.plan, share) == 0
        A, P = S.pack_aux(aux), S.pack_paths(paths)
        for s in range(8):
            S.sweep(A, P, s, 1)
            assert S.status() == (0, -1), s
            if share:
                phases.append(fhmc.fh_debug_staged(S.plan)[1:])
                assert torch.equal(P, got[s][0]) and torch.equal(A, got[s][1]), s
            else:
                got[s] = P.clone(), A.clone()
        S.close()
    slots, _, tasks, in_a, in_b, ran = phases[0]
    # (FFT plans share filters in phase A only, so nothing is listed before a chain is held)
    assert slots == (0 if prec == "fp32" else 4 * nb) and (tasks > 0) == (slots > 0) and in_a == 0
    if prec == "mfma3" and L > 32:
        assert in_b == 1 and ran == 2 * nb  # one recursion per spin and block
    else:
        assert in_b == 0 and ran == 0
    assert any(p[3] > 0 and p[2] > 0 for p in phases[1:]), phases  # phase A, with staged slots
