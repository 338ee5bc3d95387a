"""A filled filter row is the row its worldline reads, shared or its own: fh_get_filters returns the
filled values for it and for the worldlines that share it, and its draw fails on a row of zeros."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_a_filled_row_is_the_one_its_worldline_reads(prec):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    d = synth.ChainDesc(L=12, L_tau=11, n_up=10, n_dn=9, hs_kind=synth.HS_HIRSCH, block_len=4, t=1.0,
                        U=4.0, dtau=0.05, seed=5)
    print("filled rows", prec, flush=True)
    S = Sampler([d], precision)
    A = S.pack_aux([synth.initial_aux(d)])
    P = S.pack_paths([np.repeat(synth.random_walk_paths(d, 2)[:, [0, 10]], [10, 9], axis=1)])
    S.forward_filter(A, P, 0)
    rep = fhmc.fh_debug_representatives(S.plan).reshape(19, 3)
    assert np.all(rep[:10] == 0) and np.all(rep[10:] == 10)
    before = S.filters(0, 7)
    for row in (0, 4, 7):  # one of each block (3, 3 and 2 rows)
        assert fhmc.lib.fh_debug_fill_filter_row(S.plan, 0, 7, row, 0.0) == 0
    for p in (7, 0):
        got = S.filters(0, p)
        assert np.all(got[[0, 4, 7]] == 0.0)
        assert np.array_equal(np.delete(got, [0, 4, 7], 0), np.delete(before, [0, 4, 7], 0))
    assert np.all(S.filters(0, 12) > 0.0)
    if prec == "fp64":
        S.backward_sample(P, 0)
        assert S.status() == (fhmc.FH_ERR_ZERO_WEIGHT, 0)
    S.logz_grad(A, P, 0)
    assert fhmc.lib.fh_debug_fill_filter_row(S.plan, 0, 14, 3, 0.25) == 0
    assert np.all(S.filters(0, 14)[3] == 0.25) and np.all(S.filters(0, 18)[3] == 0.25)
    assert not np.any(S.filters(0, 3)[3] == 0.25)
    S.close()
