"""The one-launch random orders (up to 4096 peers) against the oracle: permutations, chunk-index
keys over many rounds with failures (keys with more than M and with no members), and rounds in
random groups with a mask."""
import numpy as np
import pytest
import torch

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
