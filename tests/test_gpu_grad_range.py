"""The FP32 adjoint of a ring shared by a thousand worldlines is finite wherever that of one worldline
would be with backward messages of mass 1: down to overlaps <f, beta> of the spin's coefficient over
FP32's largest value, a thousand times smaller than the shared factor's own limit; and it is a thousand
times the one's."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def overlaps(fhmc, d, aux, a, e):
    """The smaller of <f_j, beta_j>, j = 0, 1, of the ring a -> e over two slices from slice 0, with
    rows and messages of mass 1, in FP64."""
    g = np.zeros(d.L)
    assert fhmc.lib.fh_debug_kernel_table(d.L, d.t, d.dtau,
                                          g.ctypes.data_as(ctypes.POINTER(ctypes.c_double))) == 0
    C = g[(np.arange(d.L)[:, None] - np.arange(d.L)[None, :]) % d.L]
    conv = lambda f: C @ f @ C  # noqa: E731
    at = lambda s: np.eye(1, d.N, s).reshape(d.L, d.L)  # noqa: E731
    lam = np.arccosh(np.exp(d.dtau * d.U / 2))
    W = np.exp(lam * aux[1]).reshape(d.L, d.L)
    f1, beta1 = conv(at(a)) * W, conv(at(e))
    u1 = beta1 * W
    return min((f1 / f1.sum() * beta1).sum(), (conv(u1 / u1.sum()) * at(a)).sum()), lam


def test_shared_gradients_are_finite_where_single_ones_are():
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    L, n, near, far = 24, 1000, 0, 0
    print("gradient range", flush=True)
    for dx in range(0, 13, 2):
        for dy in range(0, 13):
            a, e = 0, dx + L * dy  # half of the worldlines runs a -> e, the other half e -> a
            got = {}
            for m in (1, n):
                d = synth.ChainDesc(L=L, L_tau=2, n_up=2 * m, n_dn=0, hs_kind=1, block_len=0, t=1.0,
                                    U=4.0, dtau=0.02, seed=1)
                aux = synth.initial_aux(d)
                S = Sampler([d], fhmc.FH_FP32_MFMA3)
                S.set_permutation([np.arange(2 * m).reshape(2, m)[::-1].ravel()])
                row = np.repeat([a, e], m).astype(np.int32)
                got[m] = S.logz_grad(S.pack_aux([aux]), S.pack_paths([np.tile(row, (2, 1))]),
                                     0)[1].cpu().numpy()
                S.close()
            (x, lam), (y, _) = overlaps(fhmc, d, aux, a, e), overlaps(fhmc, d, aux, e, a)
            if min(x, y) < 1.01 * lam / 3.4e38:
                continue
            assert np.all(np.isfinite(got[n])), (dx, dy)
            assert np.linalg.norm(got[n] - n * got[1]) <= 1e-3 * np.linalg.norm(got[n]), (dx, dy)
            near += 1
            far += min(x, y) < n * lam / 3.4e38
    assert near > 40 and far > 0, (near, far)  # the range between the two limits was met
