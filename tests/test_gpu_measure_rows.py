"""Equal-time observables of small plans, whose rows the last kernel adds by itself, have the bits they
have beside a chain whose rows take a kernel of their own: at the line (16 slices, 256 sites), below it
and above it."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,L_tau", [(2, 2), (4, 3), (4, 16), (9, 15), (16, 16), (16, 17), (18, 16)])
def test_observables_alone_and_beside_a_long_chain(L, L_tau):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    n = max(1, L * L // 2)
    d = synth.ChainDesc(L=L, L_tau=L_tau, n_up=n, n_dn=max(1, n - 1), hs_kind=1, block_len=0, t=1.0,
                        U=4.0, dtau=0.05, seed=2)
    longer = synth.ChainDesc(L=24, L_tau=40, n_up=9, n_dn=5, hs_kind=1, block_len=0, t=1.0, U=4.0,
                             dtau=0.05, seed=3)
    print("observables", L, L_tau, flush=True)
    paths = [synth.random_paths(d, 1), synth.random_paths(longer, 2)]
    S, B = Sampler([d], fhmc.FH_FP64), Sampler([d, longer], fhmc.FH_FP64)
    one, both = S.measure(S.pack_paths(paths[:1])), B.measure(B.pack_paths(paths))
    assert S.status() == B.status() == (0, -1)
    for x, y in zip(one[0], both[0]):
        assert np.array_equal(x, y)
    S.close()
    B.close()
