"""The FP64 adjoint of a chain is the same bits whatever else is in its plan: alone (one tile for
L <= 16, the 2 x 2 tiling above), and in a plan that holds both kinds, with checkpoints and without."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 16])
@pytest.mark.parametrize("small,large", [(16, 18), (4, 32), (2, 24)])
def test_fp64_adjoint_in_plans_of_one_and_of_both_tilings(small, large, flags):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    # more start sites than rings that get a workgroup of their own
    descs = [synth.ChainDesc(L=L, L_tau=9, n_up=L * L, n_dn=max(1, L * L // 3), hs_kind=1,
                             block_len=0, t=1.0, U=4.0, dtau=0.05, seed=L) for L in (small, large)]
    print("adjoint tilings", small, large, flags, flush=True)
    aux = [synth.initial_aux(d) for d in descs]
    paths = [synth.random_walk_paths(d, 3) for d in descs]

    def grads(which):
        S = Sampler([descs[i] for i in which], fhmc.FH_FP64, flags)
        A, P = S.pack_aux([aux[i] for i in which]), S.pack_paths([paths[i] for i in which])
        z, g, t = S.logz_grad(A, P, 4)
        assert S.status() == (0, -1)
        g = [torch.from_numpy(x) for x in S.unpack_aux(g)]
        S.close()
        return z.cpu(), g, t.cpu()

    both, lone = grads((0, 1)), [grads((0,)), grads((1,))]
    for i in (0, 1):
        assert torch.equal(both[0][i], lone[i][0][0]) and torch.equal(both[2][i], lone[i][2][0])
        assert torch.equal(both[1][i], lone[i][1][0])
