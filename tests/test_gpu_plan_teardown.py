"""Nothing writes into memory that a destroyed plan gave back: arrays that take freed blocks of many
sizes right after fh_destroy keep their values, for plans whose sweeps ran eagerly (the caller's stream
waits for the plan's side stream) and as a graph; plans made after them work."""
import time

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

MARK = 0x5A5A5A5A5A5A5A5A


@pytest.mark.parametrize("graph", [0, 1])
def test_freed_memory_stays_untouched(graph):
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    d = [synth.ChainDesc(L=32, L_tau=23, n_up=683, n_dn=1, hs_kind=1, block_len=12, t=1.0, U=4.0,
                         dtau=0.1, seed=6)]
    print("plan teardown", graph, flush=True)
    first = None
    for k in range(12):
        S = Sampler(d, fhmc.FH_FP32_MFMA3, fhmc.FH_FLAG_GRAPH if graph else 0)
        A, P = S.pack_aux([synth.initial_aux(d[0])]), S.pack_paths([synth.random_walk_paths(d[0], 3)])
        for s in range(4):
            S.sweep(A, P, s, 1)
        S.close()
        marks = [np.full(n, MARK, dtype=np.int64) for n in range(8, 512, 2) for _ in range(4)]
        time.sleep(0.02)
        for a in marks:
            assert np.all(a == MARK), (k, a.nbytes, np.flatnonzero(a != MARK))
        first = P if first is None else first
        assert torch.equal(P, first)


def test_side_streams_of_several_plans_alive_at_once():
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    d = [synth.ChainDesc(L=16, L_tau=16, n_up=60, n_dn=50, hs_kind=0, block_len=0, t=1.0, U=4.0,
                         dtau=0.02, seed=6)]
    aux = np.full((16, 256), -500.0)  # leaves FP32's range: the second sweep runs phase A
    aux[:, 136] = 0.0
    paths = np.zeros((16, 110), dtype=np.int32)
    print("plans alive at once", flush=True)
    want = None
    for _ in range(2):
        plans = [Sampler(d, fhmc.FH_FP32_MFMA3, fhmc.FH_FLAG_GRAPH * (k % 2)) for k in range(5)]
        state = [(S.pack_aux([aux]), S.pack_paths([paths])) for S in plans]
        for s in range(4):
            for S, (A, P) in zip(plans, state):
                S.sweep(A, P, s, 1)
        for S, (A, P) in zip(plans, state):
            assert S.status() == (0, -1)
            want = P if want is None else want
            assert torch.equal(P, want)
            S.close()


def test_a_refused_launch_leaves_no_error_behind():
    """The FP64 FFT adjoint of 64 x 64 takes more LDS than a workgroup has: the call says so, and the
    process's next HIP calls are not blamed for it."""
    from paper_2510_13866_amd import fhmc
    from paper_2510_13866_amd.sampler import Sampler
    d = [synth.ChainDesc(L=64, L_tau=3, n_up=2, n_dn=1, hs_kind=0, block_len=0, t=1.0, U=4.0,
                         dtau=0.05, seed=6)]
    print("refused launch", flush=True)
    S = Sampler(d, fhmc.FH_FP64)
    A, P = S.pack_aux([synth.initial_aux(d[0])]), S.pack_paths([synth.initial_paths(d[0])])
    with pytest.raises(fhmc.FhError):
        S.logz_grad(A, P, 0)
    torch.cuda.current_stream().synchronize()
    assert float((A.clone() + 1).sum() - A.sum()) == pytest.approx(A.numel(), rel=1e-9)
    S.sweep(A, P, 0, 1)
    assert S.status() == (0, -1)
    S.close()
