"""Staged backward draws (worldlines that share filter rows, drawn by one workgroup from rows in
LDS) against the full-row kernels: the same sites from the same filters and uniforms, whichever
tier decides a draw. The window's certificate is inflated to force the wider window (1e7) and the
row (infinity) on every draw."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def clustered(d, k, rng):
    """Worldlines of each spin spread unevenly over k random walks, with one long jump that no
    window covers."""
    walks = synth.random_walk_paths(synth.ChainDesc(**{**d.__dict__, "n_up": k, "n_dn": 0}),
                                    int(rng.integers(1 << 30)))
    walks[d.L_tau // 2:, 0] = (walks[d.L_tau // 2:, 0] + d.L // 2 + d.L * (d.L // 2)) % d.N
    w = rng.exponential(size=k)
    return walks[:, rng.choice(k, size=d.n_particles, p=w / w.sum())]


# the smallest lattice staged, whole and ragged workgroups of 64, more start sites than a row
# buffer holds, blocks of 1 to 6 draws (the slice loop runs four at a time), the largest rows
@pytest.mark.parametrize("L,L_tau,n_up,n_dn,block,walks", [
    (8, 9, 64, 1, 0, 1), (8, 12, 65, 63, 2, 5), (12, 10, 40, 72, 3, 20), (16, 11, 128, 130, 4, 40),
    (18, 25, 30, 200, 5, 9), (24, 12, 129, 64, 6, 70), (32, 21, 300, 257, 7, 30),
    (32, 33, 512, 100, 0, 2), (48, 7, 130, 20, 0, 3), (64, 6, 70, 65, 0, 2)])
@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_staged_draws_equal_full_row_draws(prec, L, L_tau, n_up, n_dn, block, walks):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    rng = np.random.default_rng(L + L_tau)
    descs = [synth.ChainDesc(L=L, L_tau=L_tau, n_up=n_up, n_dn=n_dn, hs_kind=k % 2,
                             block_len=block, t=1.0, U=4.0, dtau=0.05, seed=90 + k)
             for k in range(2)]
    print("staged draws", prec, L, L_tau, n_up, n_dn, block, flush=True)
    aux = [synth.initial_aux(d) for d in descs]
    paths = [clustered(d, walks, rng) for d in descs]
    perms = [np.concatenate([rng.permutation(d.n_up), d.n_up + rng.permutation(d.n_dn)])
             for d in descs]
    out = {}
    for name, flags, bound in (("full", fhmc.FH_FLAG_FULL_ROW_DRAW, 1.0), ("staged", 0, 1.0),
                               ("wide", 0, 1e7), ("row", 0, float("inf"))):
        S = Sampler(descs, precision, flags)
        assert fhmc.lib.fh_debug_inflate_window_bound(S.plan, bound) == 0
        S.set_permutation(perms)
        A, P = S.pack_aux(aux), S.pack_paths(paths)
        for s in range(3):
            P.copy_(S.pack_paths(paths))
            S.forward_filter(A, P, s)
            S.backward_sample(P, s)
            out[name, s] = P.clone()
            assert torch.equal(P, out["full", s]), (name, s)
        A, P = S.pack_aux(aux), S.pack_paths(paths)
        S.sweep(A, P, 3, 4)  # held chains of FP32 plans draw from the re-filter's FP64 rows
        out[name, "sweep"] = P
        assert torch.equal(P, out["full", "sweep"]), name
        assert S.status() == (0, -1), name
        S.close()
    assert not torch.equal(out["full", 0], out["full", 1])
