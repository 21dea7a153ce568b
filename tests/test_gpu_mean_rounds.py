"""Whole-grid passes that keep one mean per group (csrc/mean_rounds.hip) against the same rounds
taken one at a time, bit for bit, on the shapes that take them: tables in LDS and read ahead, one and two
column parts, several table registers' worth of rounds, more moves and terms than fit at hand,
more than one pass, row ends off 16 bytes, refresh, group-skip, and nobody ever absent."""
import numpy as np
import pytest
import torch

from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding
from test_gpu_grid_pass import state

pytestmark = pytest.mark.gpu


# Bytes of the whole matrix, rows a multiple of 128 bytes or not (then the matrix starts off them as well):
# from 32 MB on a failure schedule takes these passes, beyond 256 MiB (no longer in the last-level cache) tiles are wider.
LAYOUTS = {"odd": (0, False), "lines": (0, True), "34 MB": (34_000_000, False), "300 MB": (300_000_000, False),
           "300 MB lines": (300_000_000, True)}


def layout(N, P, dtype, name):
    """Row stride and offset, in elements."""
    least, lines = LAYOUTS[name]
    es = 4 if dtype == 0 else 2
    stride = max(P + 3, least // (N * es) + 5)
    return ((stride * es + 127) // 128 * 128 // es, 0) if lines else (stride | 1, 1)


def one_by_one(m, sched, presence, t0, rounds, N, M, d, curve):
    out = [m.dist_to_mean()] if curve else []
    for r in range(rounds):
        alive = None
        if sched is not None:
            if sched.refresh and r > 0:
                m.refresh(t0 + r, sched.seed, presence[r - 1], presence[r])
            alive = orc.skip_filter(N, M, d, t0 + r, presence[r]) if sched.group_skip else presence[r]
        m.round(t0 + r, alive)
        if curve:
            out.append(m.dist_to_mean())
    return np.array(out)


# M, d, P, dtype, p, rounds, refresh, group-skip, curve
FAILURES = [
    (16, 2, 259, 0, 0.05, 10, False, False, True),       # 16 terms and a few
    (16, 2, 259, 0, 0.6, 37, False, False, True),        # more terms and moves than are at hand, several registers
    (16, 2, 1_031, 1, 0.2, 70, False, False, False),     # two passes
    (16, 2, 64, 0, 0.3, 6, True, False, True),
    (8, 3, 70, 0, 0.2, 19, False, False, True),          # two column parts of 64 bytes
    (8, 3, 129, 1, 0.5, 9, True, False, False),
    (8, 3, 65, 1, 0.01, 5, False, True, False),
    (32, 2, 33, 0, 0.2, 8, False, False, False),
    (32, 2, 67, 0, 0.2, 18, True, False, False),         # registers filled twice, in both parts
    (32, 2, 70, 1, 0.1, 5, False, False, False),
    (32, 2, 45, 0, 0.1, 6, False, False, True),
    (32, 2, 45, 0, 0.003, 6, True, True, False),
    (16, 3, 8, 0, 0.2, 5, False, False, True),
    (16, 3, 23, 1, 0.1, 12, False, False, False),
    (16, 3, 17, 1, 0.7, 4, False, False, True),          # more than two moves a thread
    (16, 3, 40, 1, 0.2, 6, True, False, False),
    (16, 3, 9, 0, 0.01, 5, True, True, False),
    # many tiles: blocks of a compute unit out of step, their waves too
    (16, 2, 40_000, 0, 0.1, 6, False, False, True),
    (16, 2, 80_001, 1, 0.1, 7, False, False, False),
    (32, 2, 12_000, 0, 0.1, 6, False, False, False),
    (8, 3, 24_000, 1, 0.1, 6, False, False, False),
    (16, 3, 8_192, 0, 0.1, 5, False, False, False),
]


@pytest.mark.parametrize("M,d,P,dtype,p,rounds,refresh,skip,curve", FAILURES)
def test_with_failures(M, d, P, dtype, p, rounds, refresh, skip, curve):
    N, t0, seed = M ** d, 2, 11 + P
    print(f"mean rounds M={M} d={d} P={P} dtype={dtype} p={p} rounds={rounds} refresh={refresh} skip={skip}", flush=True)
    presence = orc.schedule_masks(2, p, seed, 2, N, t0, rounds)
    sched = binding.Schedule(kind=binding.SCHED_REJOIN, p=p, seed=seed, down_rounds=2, group_skip=skip, refresh=refresh)
    stride, offset = layout(N, P, dtype, "34 MB")
    bufA, A = state(N, P, stride, offset, dtype, seed)
    bufB, B = state(N, P, stride, offset, dtype, seed)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        want = one_by_one(m, sched, presence, t0, rounds, N, M, d, curve)
        m.bind_state(B)
        got, _ = m.run(t0, rounds, sched, want_dist=curve)
        m.sync()
    assert torch.equal(bufA, bufB)
    if curve:
        # same state, binary64 sums in another order: a few ulp per value added, times how much of s2 cancels (N at most)
        assert np.abs(got - want).max() <= 1e-11 * max(want)


@pytest.mark.parametrize("curve", [False, True])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,d,P", [(5, 3, 1_027), (6, 4, 77), (8, 4, 40), (9, 2, 515), (11, 3, 70), (12, 2, 1_025), (16, 2, 300), (16, 3, 41),
                                   (17, 1, 999), (24, 2, 130), (32, 2, 131), (7, 4, 23), (13, 3, 45)])
def test_with_everybody(M, d, P, dtype, curve):
    N, t0, rounds = M ** d, 1, 2 * d + 2
    print(f"mean rounds, nobody absent M={M} d={d} P={P} dtype={dtype}", flush=True)
    bufA, A = state(N, P, P + 1, 1, dtype, 3)
    bufB, B = state(N, P, P + 1, 1, dtype, 3)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        want = one_by_one(m, None, None, t0, rounds, N, M, d, curve)
        m.bind_state(B)
        got, _ = m.run(t0, rounds, None, want_dist=curve)
        m.sync()
    assert torch.equal(bufA, bufB)
    if curve:
        assert np.abs(got - want).max() <= 1e-11 * max(want)


@pytest.mark.parametrize("M,d,P,dtype", [(16, 2, 260, 0), (32, 2, 70, 1), (16, 3, 20, 1), (16, 3, 20, 0)])
def test_absent_peers_keep_their_nan_and_infinity_to_themselves(M, d, P, dtype):
    """Peers 3 and N - 2 hold NaN and infinities and are away until the last two rounds."""
    N, rounds = M ** d, 6
    masks = np.ones((rounds, N), dtype=np.uint8)
    masks[:4, [3, N - 2]] = 0
    sched = binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=masks)
    print(f"mean rounds, NaN M={M} d={d} P={P} dtype={dtype}", flush=True)
    stride, _ = layout(N, P, dtype, "34 MB")
    _, A = state(N, P, stride, 0, dtype, 5)
    _, B = state(N, P, stride, 0, dtype, 5)
    for X in (A, B):
        X[3, ::3] = float("nan")
        X[N - 2, 1::3] = float("inf")
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        for r in range(4):
            m.round(r, masks[r])
        m.bind_state(B)
        m.run(0, 5, binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=np.concatenate([masks[:4], np.zeros((1, N), np.uint8)])))
        m.sync()
        assert torch.isfinite(A.float()).sum() == N * P - len(range(0, P, 3)) - len(range(1, P, 3))
        assert torch.equal(A.view(torch.int32 if dtype == 0 else torch.int16), B.view(torch.int32 if dtype == 0 else torch.int16))
        m.bind_state(A)
        for r in range(rounds):
            m.round(r, masks[r])
        m.bind_state(B)
        m.run(0, rounds, sched)
        m.sync()
    # (which of several NaN a sum hands on is not laid down)
    assert torch.equal(A.isnan(), B.isnan()) and torch.equal(A.nan_to_num(7.0, 8.0, 9.0), B.nan_to_num(7.0, 8.0, 9.0))


@pytest.mark.parametrize("M,d,P,dtype,where,p,rounds,refresh", [
    (32, 2, 45, 0, "34 MB", 0.1, 23, False),             # LDS holds 10 of the sums at a time
    (32, 2, 70, 0, "300 MB lines", 0.1, 23, False),      # in two column parts
    (32, 2, 70, 0, "300 MB", 0.2, 68, True),             # and two passes
    (6, 3, 300, 1, "300 MB", 0.0, 25, False),            # 9
    (16, 2, 259, 0, "300 MB", 0.3, 30, False),           # 24 rounds a pass
])
def test_curves_of_more_rounds_than_lds_holds_sums(M, d, P, dtype, where, p, rounds, refresh):
    N, t0, seed = M ** d, 1, 5
    print(f"mean rounds, long curve M={M} d={d} P={P} dtype={dtype} {where} p={p} rounds={rounds}", flush=True)
    presence = orc.schedule_masks(1, p, seed, 0, N, t0, rounds) if p else None
    sched = binding.Schedule(kind=binding.SCHED_IID, p=p, seed=seed, refresh=refresh) if p else None
    stride, offset = layout(N, P, dtype, where)
    bufA, A = state(N, P, stride, offset, dtype, seed)
    bufB, B = state(N, P, stride, offset, dtype, seed)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        want = one_by_one(m, sched, presence, t0, rounds, N, M, d, True)
        m.bind_state(B)
        got, _ = m.run(t0, rounds, sched, want_dist=True)
        m.sync()
    assert torch.equal(bufA, bufB)
    assert np.abs(got - want).max() <= 1e-11 * max(want)
