"""Lattices between 32 and 64 without an FP64 re-filter (36 x 36, 54 x 54): past a floor of FP32's
range every later pass still computes its own filters and log Z, shared or not, and only the status
tells that the chain left the range; plans that hold no other lattices sweep."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,block", [(36, 0), (54, 3)])
def test_a_padded_chain_past_a_floor_is_filtered_every_pass(L, block):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=L, L_tau=7, n_up=9, n_dn=6, hs_kind=synth.HS_GAUSS, block_len=block,
                             t=1.0, U=4.0, dtau=0.05, seed=61),
             synth.ChainDesc(L=16, L_tau=5, n_up=4, n_dn=4, hs_kind=synth.HS_GAUSS, block_len=0,
                             t=1.0, U=4.0, dtau=0.05, seed=62)]
    print("padded chain past a floor", L, block, flush=True)
    rng = np.random.default_rng(L)
    # worldlines of a spin on three sites near the origin, one weight that counts, far from them
    sites = [np.repeat(rng.integers(0, 3, (d.L_tau, 3)), -(-d.n_particles // 3),
                       axis=1)[:, :d.n_particles] for d in descs]
    steep = [np.full((d.L_tau, d.N), -500.0) for d in descs]
    steep[0][:, (L // 2) * (L + 1)] = 0.0
    steep[1][:] = 0.0
    mild = [[synth.initial_aux(d, rng_seed=[k, d.L]) for d in descs] for k in range(6)]
    got = {}
    for share in (1, 0):
        S = Sampler(descs, fhmc.FH_FP32_MFMA3)
        assert fhmc.lib.fh_debug_share_filters(S.plan, share) == 0
        P = S.pack_paths(sites)
        S.forward_filter(S.pack_aux(steep), P, 0)
        assert S.status() == (fhmc.FH_ERR_NONFINITE, 0)  # the first chain left FP32's range
        zs, rows = [], []
        for k, aux in enumerate(mild):
            zs.append(S.forward_filter(S.pack_aux(aux), P, k))
            rows += [S.filters(0, p) for p in (0, 5, 8, 9, 14)]
            S.status()
        got[share] = torch.stack(zs), np.stack(rows)
        # a plan that never left the range
        F = Sampler(descs, fhmc.FH_FP32_MFMA3)
        for k, aux in enumerate(mild):
            assert torch.equal(zs[k], F.forward_filter(F.pack_aux(aux), P, k)), (share, k)
        assert F.status() == (0, -1)
        S.close()
        F.close()
    assert torch.equal(got[1][0], got[0][0])
    assert np.array_equal(got[1][1], got[0][1])


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("prec", ["fp32", "mfma3"])
def test_sweeps_of_a_plan_without_any_refilterable_chain(prec, graph):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=L, L_tau=7, n_up=40, n_dn=35, hs_kind=synth.HS_HIRSCH, block_len=b,
                             t=1.0, U=4.0, dtau=0.05, seed=70 + L) for L, b in ((36, 0), (54, 4))]
    print("sweeps of 36 x 36 and 54 x 54", prec, graph, flush=True)
    precision = fhmc.FH_FP32 if prec == "fp32" else fhmc.FH_FP32_MFMA3
    S = Sampler(descs, precision, fhmc.FH_FLAG_GRAPH if graph else 0)
    R = Sampler(descs, precision)
    A = S.pack_aux([synth.initial_aux(d) for d in descs])
    P = S.pack_paths([synth.random_walk_paths(d, 5) for d in descs])
    Ar, Pr = A.clone(), P.clone()
    for s in range(3):
        S.sweep(A, P, s, 1)
        R.forward_filter(Ar, Pr, s)
        R.backward_sample(Pr, s)
        R.gibbs_aux(Pr, Ar, s)
        assert S.status() == R.status() == (0, -1), s
        assert torch.equal(P, Pr) and torch.equal(A, Ar), s
    S.close()
    R.close()
