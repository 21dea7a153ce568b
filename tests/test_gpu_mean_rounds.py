"""Whole-grid passes that keep one mean per group (csrc/mean_rounds.hip) against the same rounds
taken one at a time, bit for bit, on shapes that take every instance of the kernel: tables in LDS, read ahead and as
bits, one and two column parts, streamed or not, several table registers' worth of rounds, more moves and
terms than fit at hand, more than one pass and more than one set of tables, row ends off 16 bytes,
refresh, group-skip, and nobody ever absent."""
import numpy as np
import pytest
import torch

from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding
from test_gpu_grid_pass import state

pytestmark = pytest.mark.gpu


# Bytes of the whole matrix, and whether rows are a multiple of 128 bytes (else the matrix starts off them as well): from 32 to 48 MB on
# a failure schedule takes these passes; beyond 256 MiB (no longer in the last-level cache) tiles are wider, and whole lines are streamed.
LAYOUTS = {"odd": (0, False), "lines": (0, True), "60 MB": (60_000_000, False), "300 MB": (300_000_000, False),
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


# M, d, P, dtype, where, p, rounds, refresh, group-skip, curve; where the places come from and the column parts of the
# tile (checked against the plan in test_grid_plan.py, as is that the rows of this file together take every kernel)
FAILURES = [
    (16, 2, 259, 0, "60 MB", 0.05, 10, False, False, True, "lds 1 x 128"),       # 16 terms and a few
    (16, 2, 259, 0, "300 MB", 0.4, 37, False, False, True, "lds 1 x 128"),      # more terms and moves than are at hand, several registers
    (16, 2, 256, 0, "300 MB lines", 0.1, 30, False, False, True, "lds 1 x 128"),
    (16, 2, 256, 0, "300 MB lines", 0.1, 9, True, False, False, "lds 1 x 128"),
    (16, 2, 259, 1, "300 MB lines", 0.1, 20, False, False, False, "lds 1 x 128"),
    (16, 2, 131, 0, "60 MB", 0.1, 9, False, False, False, "lds 1 x 128"),
    (16, 2, 1_031, 1, "60 MB", 0.2, 70, False, False, False, "lds 1 x 128"),     # two passes
    (16, 2, 64, 0, "60 MB", 0.2, 6, True, False, True, "lds 1 x 128"),
    (8, 3, 70, 0, "60 MB", 0.2, 19, False, False, True, "lds 1 x 64"),
    (8, 3, 129, 1, "60 MB", 0.5, 9, True, False, False, "lds 1 x 64"),
    (8, 3, 65, 1, "60 MB", 0.01, 5, False, True, False, "lds 1 x 64"),
    (8, 3, 70, 0, "60 MB", 0.1, 9, False, False, False, "lds 1 x 64"),
    # two column parts of 64 bytes: up to 8 rounds of a part are in its registers, more are fetched again for the second
    (8, 3, 70, 0, "300 MB", 0.1, 8, False, False, False, "lds 2 x 64"),
    (8, 3, 77, 0, "300 MB lines", 0.1, 19, True, False, False, "lds 2 x 64"),
    (8, 3, 70, 0, "300 MB", 0.2, 41, False, False, True, "lds 2 x 64"),
    (8, 3, 64, 0, "300 MB lines", 0.1, 70, False, False, True, "lds 2 x 64"),
    (8, 3, 129, 1, "300 MB", 0.2, 19, False, False, False, "lds 2 x 64"),
    (8, 3, 128, 1, "300 MB lines", 0.3, 20, True, False, False, "lds 2 x 64"),
    (32, 2, 33, 0, "60 MB", 0.2, 8, False, False, False, "lds 1 x 64"),
    (32, 2, 67, 0, "60 MB", 0.2, 18, True, False, False, "lds 1 x 64"),          # registers filled twice
    (32, 2, 70, 1, "60 MB", 0.1, 5, False, False, False, "lds 1 x 64"),
    (32, 2, 45, 0, "60 MB", 0.1, 6, False, False, True, "lds 1 x 64"),
    (32, 2, 45, 0, "60 MB", 0.003, 6, True, True, False, "lds 1 x 64"),
    (32, 2, 67, 0, "300 MB", 0.2, 18, True, False, False, "lds 2 x 64"),
    (32, 2, 64, 0, "300 MB lines", 0.1, 20, False, False, False, "lds 2 x 64"),
    (32, 2, 49, 0, "300 MB", 0.1, 8, False, False, True, "lds 2 x 64"),          # (the last tile has one part and a bit)
    (32, 2, 70, 1, "300 MB", 0.1, 19, False, False, False, "lds 2 x 64"),
    (32, 2, 128, 1, "300 MB lines", 0.1, 20, True, False, False, "lds 2 x 64"),
    (32, 2, 65, 1, "300 MB lines", 0.003, 9, False, True, False, "lds 2 x 64"),
    # read ahead: rows of one or two vectors
    (8, 3, 8, 0, "60 MB", 0.1, 7, False, False, False, "ahead 1 x 32"),
    (8, 3, 7, 0, "60 MB", 0.1, 9, False, False, True, "ahead 1 x 32"),
    (8, 3, 13, 1, "60 MB", 0.1, 8, True, False, False, "ahead 1 x 32"),
    (8, 3, 16, 1, "60 MB", 0.2, 7, False, False, True, "ahead 1 x 32"),
    (16, 2, 8, 0, "60 MB", 0.1, 7, False, False, False, "ahead 1 x 32"),
    (16, 2, 5, 0, "60 MB", 0.1, 8, False, False, True, "ahead 1 x 32"),
    (16, 2, 16, 1, "60 MB", 0.1, 9, True, False, False, "ahead 1 x 32"),
    (16, 2, 9, 1, "60 MB", 0.1, 7, False, False, True, "ahead 1 x 32"),
    (32, 2, 8, 0, "60 MB", 0.1, 9, False, False, False, "ahead 1 x 32"),
    (32, 2, 7, 0, "60 MB", 0.1, 7, False, False, True, "ahead 1 x 32"),
    (32, 2, 16, 1, "60 MB", 0.1, 8, False, False, False, "ahead 1 x 32"),
    (32, 2, 11, 1, "60 MB", 0.1, 9, True, False, True, "ahead 1 x 32"),
    (16, 3, 8, 0, "60 MB", 0.2, 5, False, False, True, "ahead 1 x 16"),
    (16, 3, 8, 0, "60 MB", 0.2, 5, True, False, False, "ahead 1 x 16"),
    (16, 3, 16, 1, "60 MB", 0.1, 6, False, False, True, "ahead 1 x 16"),
    (16, 3, 16, 1, "60 MB", 0.1, 7, True, False, False, "ahead 1 x 16"),
    (16, 3, 9, 0, "60 MB", 0.01, 5, True, True, False, "ahead 2 x 16"),
    (16, 3, 21, 0, "60 MB", 0.2, 8, False, False, True, "ahead 2 x 16"),
    (16, 3, 17, 1, "60 MB", 0.7, 4, False, False, True, "ahead 2 x 16"),         # more than two moves a thread
    (16, 3, 40, 1, "300 MB", 0.2, 6, True, False, False, "ahead 2 x 16"),
    # two bits a position: refilled at 16 rounds, for the second part, and a second pass
    (16, 3, 8, 0, "60 MB", 0.2, 35, False, False, False, "bits 1 x 16"),
    (16, 3, 16, 1, "60 MB", 0.1, 70, False, False, False, "bits 1 x 16"),
    (16, 3, 7, 0, "60 MB", 0.01, 12, False, True, False, "bits 2 x 16"),
    (16, 3, 23, 1, "60 MB", 0.1, 12, False, False, False, "bits 2 x 16"),
    (16, 3, 23, 1, "300 MB", 0.2, 35, False, False, False, "bits 2 x 16"),
    (16, 3, 21, 0, "60 MB", 0.1, 70, False, False, False, "bits 2 x 16"),
    # many tiles: blocks of a compute unit out of step, their waves too
    (16, 2, 40_000, 0, "60 MB", 0.1, 6, False, False, True, "lds 1 x 128"),
    (16, 2, 80_001, 1, "60 MB", 0.1, 7, False, False, False, "lds 1 x 128"),
    (32, 2, 12_000, 0, "60 MB", 0.1, 6, False, False, False, "lds 1 x 64"),
    (8, 3, 24_000, 1, "60 MB", 0.1, 6, False, False, False, "lds 1 x 64"),
    (8, 3, 150_000, 0, "300 MB", 0.1, 9, False, False, False, "lds 2 x 64"),
    (16, 3, 8_192, 0, "60 MB", 0.1, 5, False, False, False, "bits 2 x 16"),
]


@pytest.mark.parametrize("M,d,P,dtype,where,p,rounds,refresh,skip,curve,kernel", FAILURES)
def test_with_failures(M, d, P, dtype, where, p, rounds, refresh, skip, curve, kernel):
    N, t0, seed = M ** d, 2, 11 + P
    print(f"mean rounds M={M} d={d} P={P} dtype={dtype} {where} p={p} rounds={rounds} refresh={refresh} skip={skip} {kernel}", flush=True)
    presence = orc.schedule_masks(2, p, seed, 2, N, t0, rounds)
    sched = binding.Schedule(kind=binding.SCHED_REJOIN, p=p, seed=seed, down_rounds=2, group_skip=skip, refresh=refresh)
    stride, offset = layout(N, P, dtype, where)
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


# M, d, P, where, rounds, column parts in binary32
EVERYBODY = [(5, 3, 1_027, "odd", 8, "1 x 64"), (7, 3, 1_024, "lines", 8, "1 x 128"), (9, 2, 515, "odd", 6, "1 x 64"), (12, 2, 1_025, "odd", 6, "1 x 64"),
             (16, 2, 300, "odd", 6, "1 x 128"), (16, 2, 512, "lines", 7, "1 x 128"), (17, 1, 999, "odd", 4, "1 x 128"), (20, 2, 260, "lines", 6, "1 x 128"),
             (24, 2, 130, "odd", 6, "1 x 64"), (32, 2, 131, "odd", 6, "1 x 64"), (6, 4, 77, "300 MB", 10, "2 x 32"), (7, 4, 23, "odd", 10, "2 x 16"),
             (11, 3, 70, "300 MB", 8, "2 x 32"), (13, 3, 45, "300 MB", 8, None), (16, 3, 41, "odd", 8, "2 x 16"), (8, 3, 75, "300 MB", 8, "2 x 64"),
             (8, 3, 96, "300 MB lines", 8, "2 x 64"), (10, 3, 75, "300 MB", 8, "2 x 64"), (10, 3, 96, "300 MB lines", 8, "2 x 64"),
             (24, 2, 75, "300 MB", 12, "2 x 64"), (32, 2, 96, "300 MB lines", 6, "2 x 64")]


@pytest.mark.parametrize("curve", [False, True])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,d,P,where,rounds,parts", EVERYBODY)
def test_with_everybody(M, d, P, where, rounds, parts, dtype, curve):
    N, t0 = M ** d, 1
    print(f"mean rounds, nobody absent M={M} d={d} P={P} {where} dtype={dtype} {parts}", flush=True)
    stride, offset = layout(N, P, dtype, where)
    bufA, A = state(N, P, stride, offset, dtype, 3)
    bufB, B = state(N, P, stride, offset, dtype, 3)
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
    stride, _ = layout(N, P, dtype, "60 MB")
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


# M, d, P, dtype, where, p, rounds, refresh
LONG_CURVES = [
    (32, 2, 45, 0, "60 MB", 0.1, 23, False),             # LDS holds 10 of the sums at a time
    (32, 2, 70, 0, "300 MB lines", 0.1, 23, False),      # in two column parts
    (32, 2, 70, 0, "300 MB", 0.2, 68, True),             # and two passes
    (6, 3, 300, 1, "300 MB", 0.0, 25, False),            # 10 rounds a pass
    (16, 2, 259, 0, "300 MB", 0.3, 30, False),           # 24 rounds a pass
]


@pytest.mark.parametrize("M,d,P,dtype,where,p,rounds,refresh", LONG_CURVES)
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


@pytest.mark.parametrize("P,dtype,refresh", [(8, 0, False), (23, 1, False), (8, 0, True), (23, 1, True)])
def test_run_longer_than_its_tables(P, dtype, refresh):
    """16 MiB of tables hold 384 rounds of 4096 peers.  Nobody is present until shortly before they change, so that the state still differs
    from peer to peer there; the round before the change is part of the run for the refresh after it."""
    M, d, rounds, start = 16, 3, 396, 376
    N = M ** d
    print(f"mean rounds, long run P={P} dtype={dtype} refresh={refresh}", flush=True)
    masks = np.zeros((rounds, N), dtype=np.uint8)
    masks[start:] = (np.random.default_rng(rounds).random((rounds - start, N)) > 0.9).astype(np.uint8)
    masks[383:386] = (np.random.default_rng(3).random((3, N)) > 0.7).astype(np.uint8)
    stride, offset = layout(N, P, dtype, "300 MB")
    bufA, A = state(N, P, stride, offset, dtype, 12)
    bufB, B = state(N, P, stride, offset, dtype, 12)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        for t in range(rounds):
            if refresh and t > 0:
                m.refresh(t, 7, masks[t - 1], masks[t])
            m.round(t, masks[t])
        m.bind_state(B)
        m.run(0, rounds, binding.Schedule(kind=binding.SCHED_EXPLICIT, seed=7, refresh=refresh, explicit_masks=masks))
        m.sync()
    assert torch.equal(bufA, bufB)
    assert A.float().unique(dim=0).shape[0] > N // 8
