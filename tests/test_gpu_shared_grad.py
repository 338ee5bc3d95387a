"""Shared adjoints: worldlines with the same anchor and closing sites take one ring's results as
often as they share it. Against plans that hold each pair of sites once, whose results are added up
as often as the pair occurs. A sum of S terms rounded to eps each differs from S times one term by
at most S eps of the sum of magnitudes; the rings themselves round alike up to a few eps a step."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


# one tile and the 2 x 2 tiling with their edges, rings alone in a workgroup and in groups of four,
# ragged groups, no down spins, the FFT adjoint (48; rings that close on their own site: an FFT does
# not resolve the end weight of a far one), more pairs of sites than the table has keys
@pytest.mark.parametrize("L,L_tau,n_up,n_dn,sites,swap", [
    (2, 3, 5, 3, 2, False), (4, 16, 8, 8, 1, False), (9, 7, 30, 21, 4, True),
    (16, 9, 128, 60, 3, False), (16, 5, 120, 61, 60, True), (18, 6, 90, 33, 40, False),
    (32, 11, 300, 200, 2, True), (32, 8, 200, 0, 150, False), (48, 5, 20, 13, 3, False),
    (16, 2, 8600, 0, 256, True)])
@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_shared_adjoint_equals_the_sum_over_worldlines(prec, L, L_tau, n_up, n_dn, sites, swap):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    if prec == "mfma3" and (L > 32 or n_up > 1000):
        pytest.skip("the split-bf16 adjoint takes L <= 32; the table is tested once")
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    d = synth.ChainDesc(L=L, L_tau=L_tau, n_up=n_up, n_dn=n_dn, hs_kind=1, block_len=0, t=1.0,
                        U=4.0, dtau=0.05, seed=7)
    print("shared adjoint", prec, L, L_tau, n_up, n_dn, sites, swap, flush=True)
    rng = np.random.default_rng(L + sites)
    aux = synth.initial_aux(d)
    row = rng.permutation(d.N)[:sites][rng.integers(0, sites, d.n_particles)].astype(np.int32)
    perm = np.arange(d.n_particles)
    if swap:  # worldlines trade ends in pairs: a ring a -> e for every ring e -> a
        for p0, n in ((0, n_up), (n_up, n_dn)):
            perm[p0:p0 + n // 2 * 2] = perm[p0:p0 + n // 2 * 2].reshape(-1, 2)[:, ::-1].ravel()
    S = Sampler([d], precision)
    S.set_permutation([perm])
    A, P = S.pack_aux([aux]), S.pack_paths([np.tile(row, (L_tau, 1))])
    got = S.logz_grad(A, P, 1)
    assert all(torch.equal(x, y) for x, y in zip(got, S.logz_grad(A, P, 1)))
    energy = S.kinetic_energy(A, P, 1)
    assert S.status() == (0, -1)
    times = {}
    for p in range(d.n_particles):
        a, e = sorted((int(row[p]), int(row[perm[p]])))
        times[p >= n_up, a, e] = times.get((p >= n_up, a, e), 0) + 1
    keys = sorted(times)
    one = [synth.ChainDesc(L=L, L_tau=L_tau, n_up=0 if down else 1 + (a != e),
                           n_dn=1 + (a != e) if down else 0, hs_kind=1, block_len=0, t=1.0, U=4.0,
                           dtau=0.05, seed=1) for down, a, e in keys]
    R = Sampler(one, precision)
    R.set_permutation([np.arange(x.n_particles)[::-1] for x in one])
    z, g, t = (x.cpu().double().numpy() for x in R.logz_grad(
        R.pack_aux([aux] * len(keys)),
        R.pack_paths([np.tile([a, e][:x.n_particles], (L_tau, 1))
                      for (_, a, e), x in zip(keys, one)]), 1))
    assert R.status() == (0, -1)
    # a plan of two worldlines holds both directions, so it counts for two of the rings
    w = np.array([times[k] / x.n_particles for k, x in zip(keys, one)])
    z, t = w @ z, w @ t
    g = np.tensordot(w, g.reshape(len(keys), L_tau, d.N), 1)
    tol = 64 * (d.n_particles + L_tau) * 2.0 ** (-53 if prec == "fp64" else -24)
    gA = got[1].cpu().double().numpy().reshape(L_tau, d.N)
    assert abs(got[0].item() - z) <= tol * (1 + abs(z))
    assert np.linalg.norm(gA - g) <= tol * np.linalg.norm(g)
    assert abs(got[2].item() - t) <= tol * (1 + abs(t))
    assert abs(energy[0] + t / (L_tau * d.dtau)) <= tol * (1 + abs(t / (L_tau * d.dtau)))
    rows = S.filters(0, d.n_particles - 1)  # the ring it shares starts on its anchor site
    assert rows.shape == (L_tau, d.N) and np.argmax(rows[0]) == row[-1]
    S.close()
    R.close()
