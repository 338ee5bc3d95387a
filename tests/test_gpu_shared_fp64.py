"""Shared forward filters of the FP64 plans: with one recursion per start site, sweeps, log Z,
filters and draws equal those with one recursion per worldline bit for bit (the arithmetic of a
row is the same, so nothing is tolerated)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


# one tile (L <= 16: the edges of its K steps), the 2 x 2 tiling and its padding, the 16 x 16
# tilings; ragged and one-slice last blocks; few recursions (a workgroup each) and, at start
# states, more than 256 (a wavefront each)
@pytest.mark.parametrize("L,L_tau,n_up,n_dn,block,chains", [
    (2, 6, 3, 2, 0, 1), (4, 16, 8, 8, 0, 1), (8, 13, 20, 9, 4, 3), (9, 10, 11, 12, 0, 2),
    (16, 17, 128, 100, 8, 2), (18, 12, 60, 61, 0, 2), (27, 9, 40, 33, 4, 1),
    (32, 24, 300, 200, 11, 2), (48, 8, 40, 30, 0, 1), (64, 7, 30, 20, 3, 1),
    (48, 5, 150, 120, 0, 1), (64, 6, 200, 90, 3, 1)])
def test_fp64_shared_forward_filters_change_nothing(L, L_tau, n_up, n_dn, block, chains):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=L, L_tau=L_tau, n_up=n_up, n_dn=n_dn, hs_kind=k % 2,
                             block_len=block, t=1.0, U=4.0, dtau=0.05, seed=40 + k)
             for k in range(chains)]
    print("shared FP64 filters", L, L_tau, flush=True)
    S = Sampler(descs, fhmc.FH_FP64, fhmc.FH_FLAG_GRAPH)
    Sx = Sampler(descs, fhmc.FH_FP64)
    assert fhmc.lib.fh_debug_share_filters(Sx.plan, 0) == 0
    A = S.pack_aux([synth.initial_aux(d) for d in descs])
    P = S.pack_paths([synth.random_walk_paths(d, 7 + d.seed) for d in descs])
    Ax, Px = A.clone(), P.clone()
    for s in range(4):
        S.sweep(A, P, s, 1)
        Sx.sweep(Ax, Px, s, 1)
        assert S.status() == Sx.status() == (0, -1), s
        assert torch.equal(A, Ax) and torch.equal(P, Px), s
    # a clustered state: every worldline of a spin on one of three sites per slice
    for P_ in (P, Px):
        P_.copy_(S.pack_paths([np.repeat(synth.random_walk_paths(d, 3)[:, :3], -(-d.n_particles // 3),
                                         axis=1)[:, :d.n_particles] for d in descs]))
    S.permutation_update(P, 5, 2)
    Sx.permutation_update(Px, 5, 2)
    z, zx = S.forward_filter(A, P, 5), Sx.forward_filter(Ax, Px, 5)
    assert torch.equal(z, zx)
    rep = fhmc.fh_debug_representatives(S.plan)
    blocks = -(-L_tau // (block or L_tau))
    own = np.tile(np.repeat(np.arange(n_up + n_dn), blocks), chains)
    assert np.sum(rep != own) > 0 or n_up + n_dn <= 5
    for c, d in enumerate(descs):
        for p in (0, n_up - 1, n_up, d.n_particles - 1):
            assert np.array_equal(S.filters(c, p), Sx.filters(c, p)), (c, p)
    S.backward_sample(P, 5)
    Sx.backward_sample(Px, 5)
    assert S.status() == Sx.status() == (0, -1)
    assert torch.equal(P, Px)
    S.close()
    Sx.close()
