"""The sweep index of captured sweeps when calls do and do not follow one another: every call draws
with the indices it names, whatever ran on the plan before."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["FH_FP64", "FH_FP32_MFMA3"])
def test_indices_of_calls_in_any_order(gpu, precision):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    prec = getattr(fhmc, precision)
    descs = [synth.ChainDesc(L=4, L_tau=6, n_up=4, n_dn=3, hs_kind=k, block_len=0, t=1.0, U=4.0,
                             dtau=0.1, seed=5 + k) for k in range(2)]
    G = Sampler(descs, prec, fhmc.FH_FLAG_GRAPH)
    E = Sampler(descs, prec)   # a kernel sets its index before each sweep
    A = G.pack_aux([synth.initial_aux(d) for d in descs])
    P = G.pack_paths([synth.random_walk_paths(d, 3 + d.seed) for d in descs])
    Ae, Pe = A.clone(), P.clone()
    # in order, again, a gap, back, another call's index in between, the largest index, zero after it
    calls = [(0, 1), (1, 2), (3, 1), (3, 1), (9, 1), (2, 3), (5, 1), "moves", (6, 1), "swaps",
             (7, 2), (2 ** 64 - 1, 1), (0, 1), (1, 1)]
    for k, call in enumerate(calls):
        if call == "moves":
            G.local_update(A, P, 40, 1)
            E.local_update(Ae, Pe, 40, 1)
        elif call == "swaps":
            G.permutation_update(P, 41, 1)
            E.permutation_update(Pe, 41, 1)
        else:
            G.sweep(A, P, *call)
            E.sweep(Ae, Pe, *call)
        assert G.status() == E.status() == (0, -1), k
        assert torch.equal(A, Ae) and torch.equal(P, Pe), (k, call)
    G.close()
    E.close()
