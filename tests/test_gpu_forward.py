"""Split-bf16 forward recursions of the packed and padded lattices and of pairs taken apart: blocks
so short that the three W buffers do not fill, partial tiles, every lattice side with padding. The
rows agree with an FP64 plan's, and with shared filters they are the same bits as without."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

# the largest difference over the row's largest value: 5 slices of 12 products each, every one a
# sum of positive terms with relative error about 2^-22, plus its normaliser: below 1e-5
TOL = 1e-5


@pytest.mark.parametrize("sides", [(2, 3, 4, 6, 8), (9, 12, 16), (18, 24, 27), (32,),
                                   (8, 16, 24, 32)])
@pytest.mark.parametrize("L_tau,block", [(2, 0), (5, 3), (6, 0), (9, 4), (13, 7)])
def test_short_blocks_and_partial_tiles(gpu, sides, L_tau, block):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    descs = [synth.ChainDesc(L=L, L_tau=L_tau, n_up=max(1, L * L // 2 - k), n_dn=L * L // 3 + 1,
                             hs_kind=k % 2, block_len=block, t=1.0, U=4.0, dtau=0.05, seed=60 + k)
             for k, L in enumerate(sides)]
    print("forward", sides, L_tau, block, flush=True)
    S = Sampler(descs, fhmc.FH_FP32_MFMA3)
    Sx = Sampler(descs, fhmc.FH_FP32_MFMA3)
    assert fhmc.lib.fh_debug_share_filters(Sx.plan, 0) == 0
    S64 = Sampler(descs, fhmc.FH_FP64)
    aux = [synth.initial_aux(d) for d in descs]
    paths = [synth.random_walk_paths(d, 9 + d.seed) for d in descs]
    for k in range(2):
        if k == 1:  # few start sites: dense lists of representatives, pairs taken apart
            paths = [np.repeat(p[:, :5], -(-d.n_particles // 5), axis=1)[:, :d.n_particles].copy()
                     for d, p in zip(descs, paths)]
        A, P = S.pack_aux(aux), S.pack_paths(paths)
        A64, P64 = S64.pack_aux(aux), S64.pack_paths(paths)
        z, zx, z64 = S.forward_filter(A, P, 1), Sx.forward_filter(A, P, 1), S64.forward_filter(A64, P64, 1)
        assert S.status() == Sx.status() == S64.status() == (0, -1)
        assert torch.equal(z, zx)
        assert torch.allclose(z, z64, rtol=1e-5, atol=1e-4)  # a sum of at most 13 logs
        for c, d in enumerate(descs):
            for p in {0, d.n_up - 1, d.n_up, d.n_particles - 1}:
                rows, rows64 = S.filters(c, p), S64.filters(c, p)
                assert np.array_equal(rows, Sx.filters(c, p)), (k, c, p)
                if rows.size == 0:
                    continue
                rows = rows / rows.sum(axis=1, keepdims=True)
                rows64 = rows64 / rows64.sum(axis=1, keepdims=True)
                err = np.max(np.abs(rows - rows64), axis=1) / np.max(rows64, axis=1)
                assert np.max(err) <= TOL, (k, c, p)
    for s in (S, Sx, S64):
        s.close()
