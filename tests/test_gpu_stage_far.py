"""Staged backward draws from rows more than 64 GiB into a chain's filters: the sites are those of
one recursion per worldline, which reads other rows."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_staged_draws_far_into_a_large_chain():
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    # 128 KiB of rows per worldline: the down spins' first worldline lies past 64 GiB
    d = synth.ChainDesc(L=16, L_tau=64, n_up=524288 + 100, n_dn=128, hs_kind=synth.HS_GAUSS,
                        block_len=0, t=1.0, U=4.0, dtau=0.05, seed=11)
    need = d.n_particles * d.L_tau * d.N * 8 * 1.25 + (2 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %.0f GiB of device memory" % (need / 2 ** 30))
    print("staged draws past 64 GiB", flush=True)
    rng = np.random.default_rng(3)
    row = np.concatenate([rng.integers(0, 4, d.n_up), np.full(d.n_dn, 77)]).astype(np.int32)
    S = Sampler([d], fhmc.FH_FP64)
    A = S.pack_aux([synth.initial_aux(d)])
    P = torch.from_numpy(row).to("cuda:0").repeat(d.L_tau)
    P0 = P.clone()
    S.forward_filter(A, P, 0)
    S.backward_sample(P, 0)
    assert S.status() == (0, -1)
    got = P.clone()
    assert not torch.equal(got, P0)
    P.copy_(P0)
    assert fhmc.lib.fh_debug_share_filters(S.plan, 0) == 0
    S.forward_filter(A, P, 0)
    S.backward_sample(P, 0)
    assert S.status() == (0, -1)
    assert torch.equal(got, P)
    S.close()
