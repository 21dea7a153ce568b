"""Passes over a whole grid (several rounds in one call) against the same rounds taken one at a
time through moshpit_round, bit for bit: every summation shape (groups of 2 to 32, both types),
tiles in one and two column parts, row ends on every remainder of 16 bytes, rows that are not
aligned, rows shorter than a tile; failures, refresh, group-skip and explicit masks, the
distortion after every round, and the local step of Moshpit SGD."""
import time

import numpy as np
import pytest
import torch

from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding, inputs
from parity_util import TOL, assert_dist_close, dist_floor

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TD = {0: torch.float32, 1: torch.bfloat16}


def state(N, P, stride, offset, dtype, seed, scale=1.0):
    """[N, P] view at element `offset` of a buffer whose other elements hold 512."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    buf = torch.full((offset + N * stride + 16,), 512.0, dtype=TD[dtype], device=DEV)
    view = buf[offset: offset + N * stride].view(N, stride)[:, :P]
    view.copy_(torch.randn(N, P, generator=gen, device=DEV) * scale + torch.arange(N, device=DEV)[:, None] % 7)
    return buf, view


def fastest(m, call):
    """Seconds of the fastest of 8 calls, each waited for."""
    best = 1e9
    for _ in range(8):
        m.sync()
        start = time.perf_counter()
        call()
        m.sync()
        best = min(best, time.perf_counter() - start)
    return best


def cases():
    out = []
    # (M, d, P, pad, offset, dtype): one per summation shape and tile form ...
    grids = [(2, 4), (3, 3), (4, 3), (5, 3), (8, 2), (8, 3), (12, 2), (16, 2), (24, 2), (32, 2), (16, 3), (17, 1), (2, 9)]
    for k, (M, d) in enumerate(grids):
        for dtype in (0, 1):
            es = 4 if dtype == 0 else 2
            for j, extra in enumerate((0, 1, 16 // es - 1)):          # row end: whole vectors, one element over, one short
                P = (2 * 1024 if M ** d <= 64 else 300) // es * (1 + j) // (16 // es) * (16 // es) + extra
                out.append((M, d, max(P, 16 // es), (j * 3) % 5, (k + j) % 4, dtype))
    # ... and last tiles of 2 to 30 bytes next to a 1 KiB, 128- and 32-byte wide one
    for M, d, wb in ((4, 2, 128), (32, 2, 128), (16, 3, 32)):
        for left in (2, 8, 14, 16, 18, 30):
            out.append((M, d, (3 * wb + left) // 2, 0, 1, 1))
    return out


@pytest.mark.parametrize("M,d,P,pad,offset,dtype", cases())
def test_pass_equals_single_rounds(M, d, P, pad, offset, dtype):
    N, rounds, t0, seed = M ** d, 2 * d + 1, 1, 40 + P
    print(f"grid pass M={M} d={d} P={P} pad={pad} offset={offset} dtype={dtype}", flush=True)
    masks = orc.schedule_masks(2, 0.2, seed, 2, N, t0, rounds)
    sched = binding.Schedule(kind=binding.SCHED_REJOIN, p=0.2, seed=seed, down_rounds=2)
    bufA, A = state(N, P, P + pad, offset, dtype, seed)
    bufB, B = state(N, P, P + pad, offset, dtype, seed)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        want = [m.dist_to_mean()]
        for r in range(rounds):
            m.round(t0 + r, masks[r])
            want.append(m.dist_to_mean())
        m.bind_state(B)
        dist, _ = m.run(t0, rounds, sched, want_dist=True)
        assert torch.equal(bufA, bufB)
        # same state, binary64 sums in another order: a few ulp per value added, times how much of s2 cancels (N at most)
        assert np.abs(dist - np.array(want)).max() <= 1e-11 * max(want)
        m.run(t0, rounds, sched)                                     # and without the distortion
        for r in range(rounds):
            m.sync()
        m.bind_state(A)
        for r in range(rounds):
            m.round(t0 + r, masks[r])
        m.sync()
    assert torch.equal(bufA, bufB)


@pytest.mark.parametrize("M,d,P,dtype,kind,skip", [(4, 3, 1_001, 0, 1, False), (16, 3, 77, 1, 2, False), (32, 2, 130, 0, 2, True),
                                                   (8, 2, 515, 1, 3, True), (8, 2, 515, 1, 3, False), (2, 4, 9, 0, 1, False)])
def test_refresh_pass_equals_refresh_and_round(M, d, P, dtype, kind, skip):
    N, rounds, seed = M ** d, 7, 77
    print(f"refresh pass M={M} d={d} P={P} dtype={dtype} kind={kind} skip={skip}", flush=True)
    presence = orc.schedule_masks(2 if kind == 3 else kind, 0.25, seed, 2, N, 0, rounds)
    bufA, A = state(N, P, P + 3, 1, dtype, 5)
    bufB, B = state(N, P, P + 3, 1, dtype, 5)
    sched = binding.Schedule(kind=kind, p=0.25, seed=seed, down_rounds=2, group_skip=skip, refresh=True,
                             explicit_masks=presence if kind == 3 else None)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        for t in range(rounds):
            if t > 0:
                m.refresh(t, seed, presence[t - 1], presence[t])
            m.round(t, orc.skip_filter(N, M, d, t, presence[t]) if skip else presence[t])
        m.bind_state(B)
        m.run(0, rounds, sched)
        m.sync()
    assert torch.equal(bufA, bufB)


@pytest.mark.parametrize("M,d,P,pad,gpad", [(8, 2, 1_027, 0, 0), (4, 3, 999, 1, 2), (32, 2, 70, 0, 1), (16, 3, 40, 0, 0)])
def test_sgd_pass_equals_step_and_rounds(M, d, P, pad, gpad):
    N, rounds, seed = M ** d, 3, 9
    print(f"sgd pass M={M} d={d} P={P} pad={pad} gpad={gpad}", flush=True)
    masks = orc.schedule_masks(1, 0.2, seed, 0, N, 0, rounds)
    sched = binding.Schedule(kind=binding.SCHED_IID, p=0.2, seed=seed)
    bufA, A = state(N, P, P + pad, 0, 0, 3)
    bufB, B = state(N, P, P + pad, 0, 0, 3)
    _, G = state(N, P, P + gpad, 1, 0, 4)
    with binding.Moshpit(N, P, M, d, 0) as m:
        m.bind_state(A)
        m.sgd_round(0, G, 0.05, masks[0])
        for r in range(1, rounds):
            m.round(r, masks[r])
        for flags in (0, binding.RUN_FUSED):
            Y = bufB.clone()
            m.bind_state(Y[: N * (P + pad)].view(N, P + pad)[:, :P])
            dist, _ = m.sgd_run(0, rounds, G, 0.05, sched, want_dist=flags == 0, flags=flags)
            m.sync()
            assert torch.equal(bufA, Y)
    ref = orc.dist_to_mean(A.cpu().double().numpy())
    assert np.isfinite(dist if dist is not None else 0.0).all() and ref >= 0.0


@pytest.mark.parametrize("P,flags,sign", [(1_000, 0, 0), (999, binding.RUN_FUSED, 0), (1_000, binding.RUN_FUSED, -2 ** 31)])
def test_sgd_pass_zero_of_a_peer_alone_in_its_group(P, flags, sign):
    """Peers whose row and gradient are zero end their step at -0.  A round adds the rows of a group to
    +0, also a single one; a fused pass (16-byte-aligned rows) leaves a peer that is alone as it is."""
    M, d, rounds = 4, 3, 3
    N = M ** d
    print(f"sgd pass, zero of a lone peer P={P} flags={flags}", flush=True)
    masks = np.ones((rounds, N), dtype=np.uint8)
    masks[0, [9, 10, 11]] = 0                             # peer 8 is alone in round 0, and absent then
    masks[1:, 8] = 0
    X = torch.randn(N, P, device=DEV)
    X[[8, 20]] = -0.0                                     # (peer 20 has company)
    G = torch.randn(N, P, device=DEV)
    G[[8, 20]] = 0.0
    A, B = X.clone(), X.clone()
    with binding.Moshpit(N, P, M, d, 0) as m:
        m.bind_state(A)
        m.sgd_round(0, G, 0.05, masks[0])
        for r in range(1, rounds):
            m.round(r, masks[r])
        m.bind_state(B)
        m.sgd_run(0, rounds, G, 0.05, binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=masks), flags=flags)
        m.sync()
    A, B = A.view(torch.int32), B.view(torch.int32)
    assert bool((A[8] == 0).all()) and bool((B[8] == sign).all())
    A[8] = B[8]
    assert torch.equal(A, B)


@pytest.mark.parametrize("dtype", [0, 1])
def test_distortion_of_a_converged_state_with_an_outlier_first_row(dtype):
    """Row 0 (which the sums are shifted by) far from everybody else, rounds that nobody takes part in."""
    M, d, P = 8, 2, 1_001
    N = M ** d
    w = inputs.Workload("outlier", N, M, d, P, dtype, "normal", 0, 0.0, 0, 2, 21, 22)
    X = torch.ones(N, P, device=DEV).to(TD[dtype])
    X[0] = 512.0
    print(f"outlier {w}", flush=True)
    sched = binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=np.zeros((2, N), dtype=np.uint8))
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(X)
        dist, _ = m.run(0, 2, sched, want_dist=True)
    want = orc.dist_to_mean(X.cpu().double().numpy())
    assert_dist_close(dist, np.full(3, want), TOL[dtype] * 1e-3, dist_floor(P, dtype, 1.0) * 1e-3, w.name)
    assert bool((X[1:] == 1).all()) and bool((X[0] == 512).all())


@pytest.mark.parametrize("M,d,P,dtype", [(16, 3, 2_048, 1), (16, 3, 2_056, 1), (16, 3, 8_192, 0), (32, 2, 65_536, 0), (32, 2, 70_000, 0),
                                         (4, 3, 1_200_000, 0), (16, 2, 30_000, 0), (24, 2, 120_000, 0)])
def test_pass_on_either_side_of_the_size_rules(M, d, P, dtype):
    """Tile widths, parts and access kinds that change with the size of the state: 16- and 32-byte
    tiles of 4096 rows, one or two parts for 1024, states below and above 24 and 256 MiB."""
    N, rounds = M ** d, d + 1
    print(f"grid size M={M} d={d} P={P} dtype={dtype}", flush=True)
    A = torch.randn(N, P, device=DEV).to(TD[dtype])
    B = A.clone()
    masks = orc.schedule_masks(1, 0.1, 3, 0, N, 0, rounds)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        for r in range(rounds):
            m.round(r, masks[r])
        m.bind_state(B)
        m.run(0, rounds, binding.Schedule(kind=binding.SCHED_IID, p=0.1, seed=3))
        m.sync()
    assert torch.equal(A, B)


@pytest.mark.parametrize("flags", [0, binding.RUN_FUSED])
def test_zero_rounds_with_both_outputs_on_a_fresh_handle(flags):
    """No round: one distortion value and no times, also before the handle has timed anything."""
    M, d, P = 4, 2, 1_000
    N = M ** d
    X = torch.randn(N, P, device=DEV)
    before = X.clone()
    print(f"zero rounds flags={flags}", flush=True)
    sched = binding.Schedule(kind=binding.SCHED_IID, p=0.2, seed=3)
    with binding.Moshpit(N, P, M, d, 0) as m:
        m.bind_state(X)
        dist, ms = m.run(5, 0, sched, want_dist=True, want_times=True, flags=flags)
    assert dist.shape == (1,) and ms.shape == (0,) and torch.equal(X, before)
    want = orc.dist_to_mean(X.cpu().double().numpy())
    # binary64 sums of N terms per column; s2 against s1^2/N cancels by N at most
    assert abs(dist[0] - want) <= 4 * N * N * 2.0 ** -53 * want


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,d,P,rounds", [(16, 3, 24, 30), (2, 11, 8, 15), (8, 4, 16, 25), (4, 2, 504, 130), (32, 2, 40, 131)])
def test_run_of_several_passes(M, d, P, rounds, dtype):
    """More rounds than one pass takes (11 to 64), and not a multiple of the axes: plain, with refresh,
    group-skip and both, and as an iteration of Moshpit SGD, each against its rounds one at a time; and
    the curve.  Few peers take part, and in long runs only next to the rounds where a pass can end, so that
    the state differs from peer to peer to the end."""
    N, t0, seed = M ** d, 1, 33
    print(f"several passes M={M} d={d} P={P} rounds={rounds} dtype={dtype}", flush=True)
    rng = np.random.default_rng(rounds)
    masks = (rng.random((rounds, N)) < 0.12).astype(np.uint8)
    for r in range(rounds):
        if rounds > 64 and (r + 2) % 64 > 3:
            masks[r] = 0
        if r not in (0, 14, 64):
            continue
        S = M ** ((t0 + r) % d)                            # a whole group, for group-skip
        g = int(rng.integers(N // M))
        masks[r, (g // S) * S * M + g % S + S * np.arange(M)] = 1
    _, X = state(N, P, P, 0, dtype, 6, 3.0)
    _, G = state(N, P, P, 0, dtype, 7)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        for kind in ("plain", "refresh", "skip", "refresh skip", "sgd", "sgd refresh"):
            refresh, skip = "refresh" in kind, "skip" in kind
            live = [orc.skip_filter(N, M, d, t0 + r, masks[r]) if skip else masks[r] for r in range(rounds)]
            A, B = X.clone(), X.clone()
            m.bind_state(A)
            want = [m.dist_to_mean()]
            for r in range(rounds):
                if refresh and r > 0:
                    m.refresh(t0 + r, seed, masks[r - 1], masks[r])
                if "sgd" in kind and r == 0 and (dtype == 0 or refresh):
                    m.sgd_round(t0, G, 0.05, live[0])
                else:
                    if "sgd" in kind and r == 0:           # a fused bfloat16 pass rounds the step
                        m.local_step(G, 0.05, live[0])
                    m.round(t0 + r, live[r])
                want.append(m.dist_to_mean())
            sched = binding.Schedule(kind=binding.SCHED_EXPLICIT, seed=seed, refresh=refresh, group_skip=skip, explicit_masks=masks)
            flags = binding.RUN_FUSED if kind == "sgd" else 0
            m.bind_state(B)
            dist = None
            if "sgd" in kind:
                dist, _ = m.sgd_run(t0, rounds, G, 0.05, sched, want_dist=True, flags=flags)
            else:
                dist, _ = m.run(t0, rounds, sched, want_dist=True)
            assert torch.equal(A, B), kind
            have = ~np.isnan(dist)
            assert have[0] and have[-1] and (flags != 0 or have.all())
            # binary64 sums in another order: a few ulp per value added, times how much of s2 cancels
            assert np.abs(dist - np.array(want))[have].max() <= 1e-11 * max(want), kind
            if "sgd" not in kind:
                B.copy_(X)
                m.run(t0, rounds, sched)                   # and without the distortion
                m.sync()
                assert torch.equal(A, B), kind
            if not refresh:                                # (a refresh makes rows equal)
                assert A.float().unique(dim=0).shape[0] > N // 4, kind


@pytest.mark.parametrize("M,d,P,dtype,rounds,refresh", [(16, 3, 24, 1, 962, True), (2, 11, 8, 0, 4_104, False)])
def test_run_longer_than_its_tables(M, d, P, dtype, rounds, refresh):
    """More rounds than the tables of a pass are built for at once.  Nobody is present until shortly
    before the tables change, so that the state still differs from peer to peer there."""
    N, start = M ** d, (946 if refresh else 4_080)          # the tables change at round 952 (4,092)
    print(f"long run M={M} d={d} rounds={rounds} refresh={refresh}", flush=True)
    masks = np.zeros((rounds, N), dtype=np.uint8)
    masks[start:] = (np.random.default_rng(rounds).random((rounds - start, N)) > 0.9).astype(np.uint8)
    bufA, A = state(N, P, P, 0, dtype, 12)
    bufB, B = state(N, P, P, 0, dtype, 12)
    with binding.Moshpit(N, P, M, d, dtype) as m:
        m.bind_state(A)
        for t in range(start, rounds):
            if refresh:
                m.refresh(t, 7, masks[t - 1], masks[t])
            m.round(t, masks[t])
        m.bind_state(B)
        m.run(0, rounds, binding.Schedule(kind=binding.SCHED_EXPLICIT, seed=7, refresh=refresh, explicit_masks=masks))
        m.sync()
        assert torch.equal(bufA, bufB)
        if not refresh:                       # the same length with drawn failures: groups of two that rarely meet
            masks = orc.schedule_masks(1, 0.99, 5, 0, N, 3, rounds)
            m.bind_state(A)
            for r in range(rounds):
                m.round(3 + r, masks[r])
            m.bind_state(B)
            m.run(3, rounds, binding.Schedule(kind=binding.SCHED_IID, p=0.99, seed=5))
            m.sync()
            assert torch.equal(bufA, bufB)
    assert A.float().unique(dim=0).shape[0] > 1


@pytest.mark.parametrize("kind,skip", [(1, False), (1, True), (2, False), (2, True), (3, True)])
def test_bf16_step_then_passes(kind, skip):
    """A bfloat16 iteration without RUN_FUSED: its first round is the single-round kernel's, which
    sees the first round's mask after the group-skip filter; the passes after it see the presence."""
    M, d, P, t0, rounds, seed = 4, 3, 333, 2, 5, 21
    N = M ** d
    print(f"bf16 step kind={kind} skip={skip}", flush=True)
    presence = orc.schedule_masks(2 if kind == 3 else kind, 0.1, seed, 2, N, t0, rounds)
    bufA, A = state(N, P, P, 0, 1, 3)
    bufB, B = state(N, P, P, 0, 1, 3)
    _, G = state(N, P, P, 0, 1, 4)
    masks = [orc.skip_filter(N, M, d, t0 + r, presence[r]) if skip else presence[r] for r in range(rounds)]
    sched = binding.Schedule(kind=kind, p=0.1, seed=seed, down_rounds=2, group_skip=skip, refresh=True,
                             explicit_masks=presence if kind == 3 else None)
    with binding.Moshpit(N, P, M, d, 1) as m:
        m.bind_state(A)
        m.sgd_round(t0, G, 0.05, masks[0])
        for r in range(1, rounds):
            m.refresh(t0 + r, seed, presence[r - 1], presence[r])
            m.round(t0 + r, masks[r])
        m.bind_state(B)
        m.sgd_run(t0, rounds, G, 0.05, sched)
        m.sync()
    assert torch.equal(bufA, bufB)


def test_scratch_of_a_curve_does_not_grow_with_its_rounds():
    """600 distortions of a state of 256 MiB in 524,288 tiles: the sums of all rounds would take 2.5 GB,
    those of a pass are held to 256 MiB (63 rounds).  Every entry against the same rounds asked for in other pieces."""
    M, d, P, rounds = 2, 1, 1 << 25, 600
    N = M ** d
    print("scratch of a curve", flush=True)
    A = torch.randn(N, P, device=DEV)
    B = A.clone()
    masks = orc.schedule_masks(1, 0.9, 8, 0, N, 0, rounds)      # (two peers, both present once in 100 rounds)
    sched = binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=masks)
    with binding.Moshpit(N, P, M, d, 0) as m:
        m.bind_state(A)
        m.run(0, 1, None)                                        # (what any run allocates)
        A.copy_(B)
        m.sync()
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        dist, _ = m.run(0, rounds, sched, want_dist=True)
        assert free - torch.cuda.mem_get_info()[0] <= (256 + 16) << 20         # (16 MiB: the other outputs and masks)
        m.bind_state(B)
        first, pieces = 0, []
        for part in (1, 63, 64, 65, 200, 207):
            some = binding.Schedule(kind=binding.SCHED_EXPLICIT, explicit_masks=masks[first: first + part])
            piece, _ = m.run(first, part, some, want_dist=True)
            pieces += list(piece if first == 0 else piece[1:])
            first += part
        assert first == rounds and torch.equal(A, B)
        assert np.array_equal(dist, np.array(pieces))
        want = m.dist_to_mean()
    assert dist[0] > 0.0 and abs(dist[-1] - want) <= 1e-11 * dist[0]


def test_fused_curve_computes_only_what_it_returns():
    """Ten rounds under RUN_FUSED return the first and the last distortion: the run must cost no more
    than the rounds and two distortions on their own (a quarter allowed for the spread of timings;
    computing all eleven takes half as long again)."""
    M, d, P, rounds = 16, 2, 1_048_576, 10
    print("cost of a fused curve", flush=True)
    X = torch.randn(M ** d, P, device=DEV)
    sched = binding.Schedule(kind=binding.SCHED_IID, p=0.05, seed=3)
    with binding.Moshpit(M ** d, P, M, d, 0) as m:
        m.bind_state(X)
        dist, _ = m.run(0, rounds, sched, want_dist=True, flags=binding.RUN_FUSED)
        assert not np.isnan(dist[[0, -1]]).any() and np.isnan(dist[1:-1]).all()
        curve = fastest(m, lambda: m.run(0, rounds, sched, want_dist=True, flags=binding.RUN_FUSED))
        plain = fastest(m, lambda: m.run(0, rounds, sched, flags=binding.RUN_FUSED))
        alone = fastest(m, m.dist_to_mean)
    print(f"  curve {1e6 * curve:.0f} us, rounds {1e6 * plain:.0f}, a distortion {1e6 * alone:.0f}", flush=True)
    assert curve <= 1.25 * (plain + 2 * alone)


@pytest.mark.parametrize("M,d,P,dtype,rounds,p,skip", [(16, 3, 262_144, 1, 2, 0.2, False), (32, 2, 524_288, 0, 8, 0.2, True),
                                                       (16, 2, 1_048_576, 0, 2, 0.9, False), (7, 4, 131_072, 1, 2, 0.0, False)])
def test_run_costs_no_more_than_its_rounds_one_by_one(M, d, P, dtype, rounds, p, skip):
    """Runs that whole-grid passes would take 1.4 to 2 times as long for: few rounds on tall grids, hardly
    anybody averaged.  (A quarter and a launch allowed for the spread of timings.)"""
    print(f"cost of a run M={M} d={d} rounds={rounds} p={p} skip={skip}", flush=True)
    X = torch.randn(M ** d, P, device=DEV).to(TD[dtype])
    sched = binding.Schedule(kind=binding.SCHED_IID, p=p, seed=3, group_skip=skip) if p > 0 else None
    masks = orc.schedule_masks(1, p, 3, 0, M ** d, 0, rounds) if p > 0 else None
    if skip:
        masks = np.stack([orc.skip_filter(M ** d, M, d, t, masks[t]) for t in range(rounds)])

    def one_by_one():
        for t in range(rounds):
            m.round(t, None if masks is None else masks[t])

    with binding.Moshpit(M ** d, P, M, d, dtype) as m:
        m.bind_state(X)
        run = fastest(m, lambda: m.run(0, rounds, sched))
        alone = fastest(m, one_by_one)
    print(f"  run {1e6 * run:.0f} us, its rounds {1e6 * alone:.0f}", flush=True)
    assert run <= 1.25 * alone + 20e-6
