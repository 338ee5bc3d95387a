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


def test_the_first_call_takes_one_set_of_rows():
    import torch
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    d = synth.ChainDesc(L=64, L_tau=4096, n_up=1, n_dn=0, hs_kind=1, block_len=2048, t=1.0, U=4.0,
                        dtau=0.05, seed=2)
    print("rows of the observables", flush=True)
    S = Sampler([d], fhmc.FH_FP32_MFMA3)
    P = S.pack_paths([synth.initial_paths(d)])
    out = [torch.empty(k, dtype=torch.float64, device="cuda:0") for k in (4096, 4096, 1, 1)]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    fhmc.fh_measure(S.plan, P, *out)
    torch.cuda.synchronize()
    rows = 8 * (d.L_tau * d.N + 2 * d.L_tau)  # 128 MiB
    assert free - torch.cuda.mem_get_info()[0] <= rows + (16 << 20)
    assert S.status() == (0, -1)
    S.close()
