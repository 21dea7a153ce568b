"""Rounds that deal their work items to the dies in runs (rows off the cache lines, states too large for the last-level cache): every
work item once, for fewer of them than dies, no whole run, whole runs and a rest, and every rule of waves and accesses,
against the plain order, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2103_03239_amd import binding
from test_gpu_grid_pass import state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,d,P,MB", [(2, 3, 1_001, 480), (3, 4, 257, 480), (4, 3, 16_001, 480), (5, 2, 129, 480), (5, 3, 2_051, 900),
                                      (8, 2, 1_025, 480), (8, 2, 33_001, 900), (16, 2, 4_097, 480), (17, 2, 2_501, 480),
                                      (32, 2, 4_099, 480), (40, 2, 1_003, 480), (16, 3, 515, 480)])
def test_every_work_item_once(M, d, P, MB, dtype, masked):
    N, es = M ** d, 4 if dtype == 0 else 2
    stride = MB * 1_000_000 // (N * es) | 1
    bufA, A = state(N, P, stride, 1, dtype, P)
    bufB, B = state(N, P, stride, 1, dtype, P)
    alive = (np.random.default_rng(P).random(N) >= 0.1).astype(np.uint8) if masked else None
    print(f"runs M={M} d={d} P={P} of {MB} MB dtype={dtype} masked={masked}", flush=True)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        for X, order in ((A, 0), (B, -1)):
            m.bind_state(X)
            m.set_tuning(order=order)
            for t in range(d):
                m.round(t, alive)
        m.sync()
    assert torch.equal(bufA, bufB)


# (140,001 columns of 16 x 16 peers: more work items than blocks of a part-filled list)
@pytest.mark.parametrize("call", ["chunks", "random", "sgd"])
@pytest.mark.parametrize("M,d,P,dtype", [(16, 2, 140_001, 0), (16, 2, 280_001, 1), (4, 3, 1_027, 0), (8, 3, 259, 1), (32, 2, 4_099, 0)])
def test_peer_lists_and_local_steps(M, d, P, dtype, call):
    N, es = M ** d, 4 if dtype == 0 else 2
    stride = 480_000_000 // (N * es) | 1
    bufA, A = state(N, P, stride, 1, dtype, P)
    bufB, B = state(N, P, stride, 1, dtype, P)
    _, G = state(N, P, P + 1, 1, dtype, P + 1)
    alive = (np.random.default_rng(P).random(N) >= 0.1).astype(np.uint8)
    print(f"runs {call} M={M} d={d} P={P} dtype={dtype}", flush=True)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        for X, order in ((A, 0), (B, -1)):
            m.bind_state(X)
            m.dynamic_reset()
            m.set_tuning(order=order)
            for t in range(3):
                if call == "chunks":
                    m.dynamic_round(t, 7, alive)
                elif call == "random":
                    m.random_groups_round(t, 7, M, alive)
                else:
                    m.sgd_round(t, G, 0.05, alive)
        m.sync()
    assert torch.equal(bufA, bufB)
