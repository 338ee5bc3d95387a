"""Equal-time observables with two slices per transform and slice sums split over workgroups, at
the sizes where a split has remainders, against the oracle's direct sums."""
import numpy as np
import pytest

import synth
from oracle import measure as omeasure

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shapes", [
    [(2, 2), (64, 3), (3, 17), (6, 33), (9, 16), (27, 2), (48, 15)],   # odd, even, one tile, many
    [(36, 5)], [(2, 3)], [(54, 7), (4, 1030)]])
def test_pairs_and_tiles(gpu, shapes):
    """S(k), C(r) within 1e-12 of their largest value (FP64 transforms of length below 100: about
    20 roundings of 1.1e-16), D and the local moment (whole numbers over n) to 1e-14; the same bits
    twice; worldlines outnumber the sites on the smallest lattice."""
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=L, L_tau=l_tau, n_up=L * L // 2 + 3, n_dn=L * L // 3 + 1,
                             hs_kind=synth.HS_HIRSCH, block_len=0, t=1.0, U=4.0, dtau=0.1, seed=i)
             for i, (L, l_tau) in enumerate(shapes)]
    rng = np.random.default_rng(len(shapes))
    paths = [rng.integers(0, d.N, size=(d.L_tau, d.n_particles)).astype(np.int32) for d in descs]
    S = Sampler(descs, fhmc.FH_FP64)
    P = S.pack_paths(paths)
    got, again = S.measure(P), S.measure(P)
    assert S.status() == (0, -1)
    for c, d in enumerate(descs):
        ref = omeasure.observables(d.L, d.n_up, paths[c])
        for i in (0, 1):
            assert np.max(np.abs(got[c][i] - ref[i])) <= 1e-12 * max(1.0, np.max(np.abs(ref[i])))
            assert np.array_equal(got[c][i], again[c][i])
        for i in (2, 3):
            assert got[c][i] == pytest.approx(ref[i], rel=1e-14, abs=1e-300)
    S.close()
