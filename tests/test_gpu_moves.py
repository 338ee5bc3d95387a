"""Local moves of the end slices and reconnection swaps at their smallest shapes, against the
oracle: two-slice rings (whose slice 1 neighbours slice 0 on both sides) beside longer ones, and
many small chains within one wavefront. Sites and permutations are equal; a worldline may differ
only where the oracle certifies a near-tie (|u - R| < 1e-9)."""
import numpy as np
import pytest

import synth
from oracle import local as olocal, perm as operm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("taus", [(2,), (3,), (2, 3, 4, 5, 2), (7, 8, 9, 10, 130)])
def test_end_slice_moves_with_reconnections(taus):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=(3, 4, 6, 8, 9)[i], L_tau=t, n_up=7 + 60 * (i % 2), n_dn=5, hs_kind=i % 2,
                             block_len=0, t=1.0, U=4.0, dtau=0.3, seed=20 + i)
             for i, t in enumerate(taus)]
    print("end slice moves", taus, flush=True)
    S = Sampler(descs, fhmc.FH_FP64)
    rng = np.random.default_rng(5)
    perms = [np.concatenate([rng.permutation(d.n_up), d.n_up + rng.permutation(d.n_dn)])
             for d in descs]
    S.set_permutation(perms)
    aux = [synth.initial_aux(d) for d in descs]
    paths = [synth.random_walk_paths(d, 30 + d.seed) for d in descs]
    A, P = S.pack_aux(aux), S.pack_paths(paths)
    S.local_update(A, P, 6, 3)
    assert S.status() == (0, -1)
    got = S.unpack_paths(P)
    for c, d in enumerate(descs):
        ref, margins = olocal.local_update(d, aux[c], paths[c], 6, 3, True, perm=perms[c])
        assert margins.min() > 1e-9, c  # no near-tie at these seeds
        assert np.array_equal(got[c], ref), c
        assert (got[c][[0, -1]] != paths[c][[0, -1]]).any(), c
    S.close()


@pytest.mark.parametrize("sizes", [(2, 3, 1, 4, 2, 2), (64, 63, 65), (130,)])
def test_swaps_of_many_chains_in_a_wavefront(sizes):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=4, L_tau=4, n_up=n, n_dn=n // 2, hs_kind=0, block_len=0, t=1.0,
                             U=4.0, dtau=0.5, seed=60 + i) for i, n in enumerate(sizes)]
    print("swaps", sizes, flush=True)
    S = Sampler(descs, fhmc.FH_FP64)
    paths = [synth.random_walk_paths(d, 70 + d.seed) for d in descs]
    paths[0][:] = paths[0][:, :1]  # every worldline on one path: every swap is accepted
    P = S.pack_paths(paths)
    S.permutation_update(P, 9, 5)
    got, sign = S.permutation()
    for c, d in enumerate(descs):
        ref, flips, margins = operm.perm_update(d, paths[c], np.arange(d.n_particles), 9, 5, True)
        assert min([m.min() for m in margins if len(m)] or [1.0]) > 1e-9, c
        assert np.array_equal(got[c], ref), c
        assert sign[c] == (-1) ** flips, c
    S.close()
