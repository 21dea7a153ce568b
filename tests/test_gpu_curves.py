"""Distortions inside a whole-grid pass where their split over threads has edges: fewer threads than 4-byte words of a row, as many, threads
left over, one and several row parts, odd numbers of waves, a last tile of a few bytes; against binary64 sums over the states of the same
rounds taken one at a time."""
import numpy as np
import pytest
import torch

from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding
from test_gpu_grid_pass import state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [0.0, 0.2])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,d,bytes_", [
    (2, 1, 2_064), (2, 2, 1_020), (3, 2, 4_100), (24, 1, 2_050),     # 64 to 192 threads, rows of 256 words
    (27, 1, 1_032), (2, 5, 3_080),                                   # as many threads as words
    (6, 2, 1_546), (7, 2, 1_028),                                    # rows of 128 words, 64 threads idle or a part more
    (3, 4, 772), (9, 2, 520), (2, 7, 1_000),                         # rows of 64 words, 3 and 4 parts
    (5, 4, 260), (3, 6, 140), (6, 3, 524), (15, 2, 390),             # shorter rows; odd numbers of waves
    (13, 3, 108), (23, 2, 1_030),                                    # 9 waves of which 3 share a distortion, 5 of which 2 do
])
def test_against_binary64(M, d, bytes_, dtype, p):
    N, rounds, t0, seed = M ** d, 2 * d + 5, 1, 11 * M + d
    P = bytes_ // (4 if dtype == 0 else 2)
    print(f"curve M={M} d={d} P={P} dtype={dtype} p={p}", flush=True)
    masks = orc.schedule_masks(1, p, seed, 0, N, t0, rounds) if p else [None] * rounds
    sched = binding.Schedule(kind=binding.SCHED_IID, p=p, seed=seed) if p else None
    bufA, A = state(N, P, P + 3, 1, dtype, seed)
    bufB, B = state(N, P, P + 3, 1, dtype, seed)
    want, scale = [], []

    def note():
        Y = A.double()
        Y = Y - Y[:1]                                                # (exact)
        want.append(float(((Y - Y.mean(0, keepdim=True)) ** 2).sum()) / N)
        scale.append(float((Y ** 2).sum()) / N)

    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        note()
        for r in range(rounds):
            m.round(t0 + r, masks[r])
            m.sync()
            note()
        m.bind_state(B)
        got, _ = m.run(t0, rounds, sched, want_dist=True)
        m.sync()
    assert torch.equal(bufA, bufB)
    # s2 and s1 are sums of N terms in binary64, of differences from row 0, and s1^2 / N <= s2
    bound = 4.0 * (N + 64) * 2.0 ** -53 * np.array(scale)
    assert (np.abs(got - np.array(want)) <= bound).all(), (got, want, bound)
