"""Single rounds, local steps, refreshes and distortions on rows that start on any element and end
on any remainder of 16 bytes: the state has the bits of the same columns in 16-byte-aligned rows
without a remainder, and nothing outside the rows is touched."""
import time

import numpy as np
import pytest
import torch

from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TD = {0: torch.float32, 1: torch.bfloat16}


def matrix(values, stride, offset):
    N, P = values.shape
    buf = torch.full((offset + N * stride + 16,), 512.0, dtype=values.dtype, device=DEV)
    view = buf[offset: offset + N * stride].view(N, stride)[:, :P]
    view.copy_(values)
    return buf, view


# M: one per default launch shape (4 columns per lane and 2 rows, 1 and 4, 2 and 8, 1 and 16, two chunks of 16);
# P: one lane short of, on and past a work item of 64, 128 or 256 vectors, rows of a few vectors and of less than one
CASES = [(M, d, P + k, dtype) for M, d, in ((2, 3), (4, 2), (7, 2), (16, 1), (20, 1))
         for dtype, P in ((0, 256), (0, 1024), (1, 512), (1, 2048), (1, 24), (0, 4)) for k in (0, 1, 3)] + \
        [(3, 2, P, dtype) for P in (1, 2, 3, 5, 7) for dtype in (0, 1)]


@pytest.mark.parametrize("M,d,P,dtype", CASES)
def test_any_row_start_and_end(M, d, P, dtype):
    N = M ** d
    pad, offset = P % 3, P % 2
    print(f"row ends M={M} d={d} P={P} dtype={dtype}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(P + M)
    per16 = 4 if dtype == 0 else 8
    wide = -(-P // per16) * per16
    full = torch.randn(N, wide, generator=gen, device=DEV).to(TD[dtype])
    grad = torch.randn(N, wide, generator=gen, device=DEV).to(TD[dtype])
    r = np.random.default_rng(P)
    alive, back = (r.random(N) > 0.2).astype(np.uint8), (r.random(N) > 0.2).astype(np.uint8)
    order = r.permutation(N)[: N - 1]
    bufA, A = matrix(full, wide, 0)                              # aligned, whole vectors
    bufB, B = matrix(full[:, :P], P + pad, offset)
    _, GA = matrix(grad, wide, 0)
    _, GB = matrix(grad[:, :P], P + (P + 1) % 3, 1 - offset)
    values = []
    for X, G, width in ((A, GA, wide), (B, GB, P)):
        with binding.Moshpit(N, width, M, d, dtype) as m:
            m.bind_state(X)
            m.round(0, alive)
            m.local_step(G, 0.1, back)
            m.sgd_round(d - 1, G, 0.05, alive)
            m.refresh(2, 5, alive, back)
            m.random_groups_round(3, 6, min(M, N - 1), alive)
            m.grouped_round(order, min(M, N - 1), back)
            values.append(m.dist_to_mean())
    assert torch.equal(A[:, :P], B)
    rest = bufB.clone()
    rest[offset: offset + N * (P + pad)].view(N, P + pad)[:, :P] = 512.0
    assert bool((rest == 512.0).all())
    want = orc.dist_to_mean(B.cpu().double().numpy())
    # binary64 sums of N terms per column: N units of 2^-53 per sum and s2 against s1^2/N cancels by N at most
    assert abs(values[1] - want) <= 4 * N * N * 2.0 ** -53 * want


@pytest.mark.parametrize("M,d,P,dtype", [(16, 2, 2_001, 0), (16, 2, 2_001, 1), (32, 2, 515, 0), (5, 5, 40, 1), (4, 7, 9, 0), (3, 1, 3, 1)])
def test_distortion_of_the_rows_that_count(M, d, P, dtype):
    """Rows are taken 64 to a wave and 8 (4) at a time, those that are left out never: with one row in
    thirty, half of them, all but one and only the last; the others hold NaN."""
    N = M ** d
    r = np.random.default_rng(N + P)
    X = torch.randn(N, P, device=DEV).to(TD[dtype])
    values = X.cpu().double().numpy()
    only_last, but_one = np.zeros(N, dtype=np.uint8), np.ones(N, dtype=np.uint8)
    only_last[-1], but_one[N // 2] = 1, 0
    for present in ((r.random(N) < 1 / 30).astype(np.uint8), (r.random(N) < 0.5).astype(np.uint8), but_one, only_last):
        present[0 if present is not only_last else -1] = 1
        print(f"distortion M={M} d={d} P={P} dtype={dtype} rows={present.sum()}", flush=True)
        Y = X.clone()
        Y[torch.from_numpy(present == 0).to(DEV)] = float("nan")
        with binding.Moshpit(N, P, M, d, dtype) as m:
            m.bind_state(Y)
            got = m.dist_to_mean_subset(present)
        rows = values[present != 0]
        want = ((rows - rows.mean(axis=0)) ** 2).sum() / len(rows)
        # binary64 sums of n terms per column; s2 against s1^2/n cancels by n at most
        assert abs(got - want) <= 8 * len(rows) ** 2 * 2.0 ** -53 * want + 1e-300


def test_distortion_keeps_its_loads_in_flight():
    """64 MB in 1024 rows that start anywhere: 62 blocks of 4 waves, each with 256 rows to walk.  One row
    at a time that takes 4.9 times as long as a copy of the state (146 us), eight at a time 2.2 (67 us)."""
    M, d, P = 32, 2, 15_625
    X = torch.randn(M ** d, P, device=DEV)
    Y = torch.empty_like(X)
    print("distortion of short rows", flush=True)

    def fastest(call):
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            start = time.perf_counter()
            call()
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - start)
        return best

    with binding.Moshpit(M ** d, P, M, d, 0) as m:
        m.bind_state(X)
        distortion, copy = fastest(m.dist_to_mean), fastest(lambda: Y.copy_(X))
    print(f"  distortion {1e6 * distortion:.0f} us, copy {1e6 * copy:.0f}", flush=True)
    assert distortion <= 3.8 * copy
