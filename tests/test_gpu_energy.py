"""The kinetic energy, whose adjoint writes no field gradient, is -(t / beta) times the d log Z / dt of
the gradient call to the rounding of that factor: the same adjoint, with and without the field
gradient and its barrier."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 16])
@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_energy_is_the_gradient_calls(prec, flags):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    descs = [synth.ChainDesc(L=L, L_tau=33, n_up=n, n_dn=n // 2, hs_kind=synth.HS_GAUSS, block_len=0,
                             t=1.0, U=4.0, dtau=0.05, seed=L) for L, n in
             ((32, 400), (27, 200), (16, 100), (9, 37), (4, 8), (2, 3))]
    print("energy", prec, flags, flush=True)
    S = Sampler(descs, precision, flags)
    A = S.pack_aux([synth.initial_aux(d) for d in descs])
    P = S.pack_paths([synth.random_walk_paths(d, 3) for d in descs])
    for anchor in (0, 5, 32):
        gt = S.logz_grad(A, P, anchor)[2].cpu().numpy()
        e = S.kinetic_energy(A, P, anchor)
        assert S.status() == (0, -1)
        beta = np.array([d.L_tau * d.dtau for d in descs])
        assert np.all(np.abs(e + gt / beta) <= 4 * 2.0 ** -53 * np.abs(e)), anchor
    S.close()
