"""Shared adjoints at the most pairs of sites that a spin shares (4096) and one more, each pair held
twice: below the line a pair's two worldlines share a ring, above it every worldline has its own, and
either way log Z, d/dt and the field gradient are twice those of the pairs held once, up to the
rounding of the sums."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def pairs_held(k, more, times):
    """Worldlines from every one of k sites to every one, `more` on a site of their own, each
    `times`: (anchor sites, permutation)."""
    a, e = (v.ravel() for v in np.meshgrid(np.arange(k), np.arange(k), indexing="ij"))
    start = np.concatenate([np.tile(a, times), np.full(more * times, k)]).astype(np.int32)
    want = np.concatenate([np.tile(e, times), np.full(more * times, k)])
    perm = np.empty(len(start), dtype=np.int64)
    perm[np.argsort(want, kind="stable")] = np.argsort(start, kind="stable")
    assert np.array_equal(start[perm], want)
    return start, perm


@pytest.mark.parametrize("k,more,shared", [(64, 0, True), (64, 1, False), (45, 0, True)])
@pytest.mark.parametrize("prec", ["fp64", "mfma3"])
def test_the_most_rings_a_spin_shares(prec, k, more, shared):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    precision = fhmc.FH_FP64 if prec == "fp64" else fhmc.FH_FP32_MFMA3
    print("many rings", prec, k, more, flush=True)
    out, aux = [], None
    for times in (1, 2):
        row, perm = pairs_held(k, more, times)
        d = synth.ChainDesc(L=16, L_tau=2, n_up=len(row), n_dn=0, hs_kind=1, block_len=0, t=1.0,
                            U=4.0, dtau=0.05, seed=3)
        S = Sampler([d], precision)
        S.set_permutation([perm])
        A = S.pack_aux([synth.initial_aux(d)])
        out.append([x.cpu().double().numpy() for x in
                    S.logz_grad(A, S.pack_paths([np.tile(row, (2, 1))]), 1)])
        assert S.status() == (0, -1)
    # the ring of a worldline and of the one that runs between the same sites
    p, q = 70, 70 + k * k
    assert row[p] == row[q] and row[perm[p]] == row[perm[q]]
    assert fhmc.lib.fh_debug_fill_filter_row(S.plan, 0, p, 1, 0.5) == 0
    assert np.all(S.filters(0, p)[1] == 0.5)
    assert np.all(S.filters(0, q)[1] == 0.5) == shared
    # sums of n terms, each of either order within n eps of the sum of magnitudes
    tol = 4 * len(row) * 2.0 ** (-53 if prec == "fp64" else -24)
    for one, two in zip(*out):
        assert np.linalg.norm(two - 2 * one) <= tol * np.linalg.norm(two)
    S.close()
