"""The one-launch random orders (up to 4096 peers) against the oracle: permutations, chunk-index
keys over many rounds with failures (keys with more than M and with no members), and rounds in
random groups with a mask."""
import os
import re
import time

import numpy as np
import pytest
import torch

import __graft_entry__ as entry
from oracle import moshpit_oracle as orc
from paper_2103_03239_amd import binding
from parity_util import assert_state_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("M,d", [(2, 1), (3, 2), (2, 10), (32, 2), (5, 5), (64, 2), (2, 12), (4, 6), (16, 3), (2, 13)])
def test_permutation_and_keys(M, d):
    N, P, seed = M ** d, 4, 17 + M
    print(f"small order M={M} d={d}", flush=True)
    r = np.random.default_rng(d)
    X = torch.rand(N, P, device=DEV) + 1.0        # positive: no sum of a group cancels
    ref = X.cpu().double().numpy().copy()
    keys = orc.dynamic_init(N, M, d)
    with binding.Moshpit(N, P, M, d, binding.F32) as m:
        m.bind_state(X)
        for t in (0, 5):
            got = m.random_permutation(t, seed)
            assert np.array_equal(got, orc.random_permutation(seed, t, N))
        for t in range(6):
            alive = None if t == 0 else (r.random(N) < (0.9, 0.5, 0.05, 1.0, 0.0)[t - 1]).astype(np.uint8)
            m.dynamic_round(t, seed, alive)
            orc.dynamic_round(ref, M, d, keys, seed, t, alive)
            assert np.array_equal(m.dynamic_keys(), np.asarray(keys).reshape(N, -1)), t
        for t, gs in ((0, M), (1, 1), (2, min(7, N))):
            alive = (r.random(N) < 0.7).astype(np.uint8)
            m.random_groups_round(t, seed, gs, alive)
            orc.grouped_round(ref, orc.random_permutation(seed, t, N), gs, alive)
        m.sync()
    # 9 rounds of at most 7 additions in a row (trees of 16, four of them) and a division, each within 2^-24
    assert_state_close(X.cpu().double().numpy(), ref, 9 * 8 * 2.0 ** -24, f"small order {M}^{d}")


@pytest.mark.parametrize("M,d", [(16, 2), (8, 3), (64, 2)])
def test_keys_that_have_come_together(M, d):
    """Rounds in which every peer is alone in its group leave it chunk 0, until all peers share one key:
    the next order ranks them among each other at about the price of any other (test_crowded_buckets has the
    grids whose buckets hold hundreds then)."""
    N, P, seed = M ** d, 4, 40 + M
    print(f"keys together M={M} d={d}", flush=True)
    r = np.random.default_rng(M)
    X = torch.rand(N, P, device=DEV) + 1.0
    ref = X.cpu().double().numpy().copy()
    keys = orc.dynamic_init(N, M, d)
    took = []
    with binding.Moshpit(N, P, M, d, binding.F32) as m:
        m.bind_state(X)

        def one_round(t, alive):
            m.sync()
            start = time.perf_counter()
            m.dynamic_round(t, seed, alive)
            m.sync()
            took.append(time.perf_counter() - start)
            orc.dynamic_round(ref, M, d, keys, seed, t, alive)
            assert np.array_equal(m.dynamic_keys(), np.asarray(keys).reshape(N, -1)), t

        t = 0
        while np.any(keys):
            flat = np.asarray(keys).reshape(N, -1) @ (M ** np.arange(d - 1))
            alive = np.zeros(N, dtype=np.uint8)
            alive[[r.choice(np.flatnonzero(flat == k)) for k in np.unique(flat[flat != 0])]] = 1
            one_round(t, alive)
            t += 1
        half = (r.random(N) < 0.5).astype(np.uint8)
        one_round(t, half)                                          # half of one bucket, then the other half
        one_round(t + 1, 1 - half)
        crowded = min(took[-2:])
        for k in (2, 3):
            one_round(t + k, None)
        apart = min(took[-2:])
    print(f"  {1e6 * crowded:.0f} us a round, {1e6 * apart:.0f} with keys apart", flush=True)
    # counting among the 2048 of a key took 240 us more
    assert crowded <= apart + 100e-6
    # at most 7 additions in a row and a division in the four rounds that average anything, each within 2^-24
    assert_state_close(X.cpu().double().numpy(), ref, 4 * 8 * 2.0 ** -24, f"keys together {M}^{d}")


def fullest_bucket(N, M, d, packed, seed, t, alive):
    """Participants of a chunk-index round in the kernel's fullest bucket: by key and as many of the order key's upper bits
    as give at most one bucket to a peer (their next power of two)."""
    def mix(x):
        x = x ^ (x >> np.uint64(32))
        x = x * np.uint64(0x9E3779B97F4A7C15)
        x = x ^ (x >> np.uint64(29))
        x = x * np.uint64(0x6A09E667F3BCC909)
        return x ^ (x >> np.uint64(32))

    with np.errstate(over="ignore"):
        order = mix(mix(np.uint64(seed) + np.uint64(0xD1B54A32D192ED03) * np.uint64(t + 1)) ^ np.arange(N, dtype=np.uint64))
    assert np.array_equal(np.argsort(order, kind="stable"), orc.random_permutation(seed, t, N))
    n_keys, most, bits = M ** (d - 1), 64, 0
    while most < N:
        most *= 2
    while n_keys << (bits + 1) <= most:
        bits += 1
    bucket = packed << bits
    if bits > 0:
        bucket = bucket + (order >> np.uint64(64 - bits)).astype(np.int64)
    return int(np.bincount(bucket[np.asarray(alive) != 0], minlength=1).max())


def crowded_from():
    """Members of a bucket above which the kernel spreads them over slots."""
    source = open(os.path.join(entry.CSRC, "small_order.hip")).read()
    return int(re.search(r"constexpr int32_t kCrowded = (\d+);", source).group(1))


# 16 x 16 x 16 and 4^6 spread 4096 peers of one key over 16 and 4 buckets, 2^12 over 2; 2^10 and 4^5 are launched with a peer to a thread
@pytest.mark.parametrize("M,d", [(16, 3), (4, 6), (2, 12), (2, 10), (4, 5)])
def test_crowded_buckets(M, d):
    """Keys come together until a bucket holds so many peers that its members are spread over slots, with all, some and few
    of them taking part; keys and the averages of every group as the oracle has them."""
    N, P, seed, limit = M ** d, 4, 90 + M, crowded_from()
    print(f"crowded M={M} d={d}", flush=True)
    r = np.random.default_rng(M + d)
    X = torch.rand(N, P, device=DEV) + 1.0
    ref = X.cpu().double().numpy().copy()
    keys = orc.dynamic_init(N, M, d)
    weights = M ** np.arange(d - 1)
    t = 0
    with binding.Moshpit(N, P, M, d, binding.F32) as m:
        m.bind_state(X)
        for share, more_than in ((1.0, limit), (0.6, limit), (0.9, max(limit, 100))):
            while True:
                packed = keys.reshape(N, -1) @ weights
                alive = (r.random(N) < share).astype(np.uint8)
                if fullest_bucket(N, M, d, packed, seed, t, alive) > more_than:
                    break
                # peers alone in their groups: each gets chunk 0 and keeps its row
                alone = np.zeros(N, dtype=np.uint8)
                some = r.permutation(np.flatnonzero(packed))
                alone[some[np.unique(packed[some], return_index=True)[1]]] = 1
                m.dynamic_round(t, seed, alone)
                keys[alone != 0] = np.pad(keys[alone != 0][:, 1:], ((0, 0), (0, 1)))
                t += 1
                assert t < 2500
            m.dynamic_round(t, seed, alive)
            orc.dynamic_round(ref, M, d, keys, seed, t, alive)
            assert np.array_equal(m.dynamic_keys(), keys.reshape(N, -1)), t
            t += 1
        m.sync()
    print(f"  3 crowded rounds of {t}", flush=True)
    # at most 7 additions in a row and a division in each of the crowded rounds, the others average nothing
    assert_state_close(X.cpu().double().numpy(), ref, 3 * 8 * 2.0 ** -24, f"crowded {M}^{d}")


@pytest.mark.parametrize("M,d,P", [(2, 3, 2_100_003), (3, 2, 2_800_000), (16, 2, 131_072)])
def test_chunk_index_rounds_of_many_work_items(M, d, P):
    """A state with so many column tiles that the launch has no blocks for the groups which fill the list's spare
    places (the blocks go on to them) against the same rounds on some of its columns, bit for bit; the masks leave
    some keys with more than M members, some with none."""
    N, seed, some = M ** d, 71 + M, 1_000
    print(f"many work items M={M} d={d}", flush=True)
    r = np.random.default_rng(M)
    X = torch.randn(N, P, device=DEV)
    parts = [X[:, :some].clone(), X[:, P // 2:P // 2 + some].clone(), X[:, P - some:].clone()]
    masks = [None] + [(r.random(N) < q).astype(np.uint8) for q in (0.6, 0.5, 0.7, 0.9, 1.0)]
    for state in [X] + parts:
        with binding.Moshpit(N, state.shape[1], M, d, binding.F32) as m:
            m.bind_state(state)
            for t, alive in enumerate(masks):
                m.dynamic_round(t, seed, alive)
            m.sync()
    for part, first in zip(parts, (0, P // 2, P - some)):
        assert torch.equal(X[:, first:first + some], part), first
