"""Sweeps at grids below and above the line from which the shared-filter map and the member pass leave
the queueing of held and of whole chains to a kernel of its own: chains that enter the FP64 re-filter,
stay on it and leave it have the same sites, fields and holds alone as in a batch on the other side."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# the map runs 2 workgroups per chain and block: 1 chain (14) against 20 (280), and the member pass
# 1 thread per worldline and block: 1 chain (7 workgroups) against 30 (210)
@pytest.mark.parametrize("n,block,copies", [(128, 5, 20), (128, 5, 30)])
def test_a_chain_alone_and_in_a_large_batch(n, block, copies):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    print("last workgroup", n, block, copies, flush=True)
    one = [synth.ChainDesc(L=16, L_tau=32, n_up=n, n_dn=n, hs_kind=synth.HS_GAUSS, block_len=block,
                           t=1.0, U=4.0, dtau=0.02, seed=5)]
    many = one + [synth.ChainDesc(**{**one[0].__dict__, "seed": 100 + k}) for k in range(copies - 1)]
    # one weight that counts, on another site than every second worldline: hops and end weights far
    # below FP32's range in the first pass, none after the field is redrawn
    aux, paths = np.full((32, 256), -500.0), synth.initial_paths(one[0])
    aux[:, 136] = 0.0
    S, B = Sampler(one, fhmc.FH_FP32_MFMA3), Sampler(many, fhmc.FH_FP32_MFMA3)
    A, P = S.pack_aux([aux]), S.pack_paths([paths])
    AB, PB = B.pack_aux([aux] * copies), B.pack_paths([paths] * copies)
    seen = []
    for s in range(24):
        S.sweep(A, P, s, 1)
        B.sweep(AB, PB, s, 1)
        assert S.status() == B.status() == (0, -1), s
        assert np.array_equal(S.unpack_paths(P)[0], B.unpack_paths(PB)[0]), s
        assert np.array_equal(S.unpack_aux(A)[0], B.unpack_aux(AB)[0]), s
        hold = fhmc.fh_debug_rescue_holds(S.plan, 1)[0]
        assert hold == fhmc.fh_debug_rescue_holds(B.plan, copies)[0], s
        seen.append(hold)
    assert max(seen) > 0 and min(seen) == 0, seen  # the chain was held, and not always
    S.close()
    B.close()
