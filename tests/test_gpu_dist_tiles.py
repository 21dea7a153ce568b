"""The distortion's pass at the edges of its tile rule: every width of a tile and number of waves it
takes, rows that end inside a vector, rows off the 16-byte boundaries, row counts that do not fill the last load."""
import pytest
import torch

from paper_2103_03239_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("N,P,dtype,odd", [
    (1, 5, 0, 1), (2, 1_000, 1, 0), (3, 4, 0, 0), (31, 70_003, 0, 1),     # fewer rows than a load takes; one wave
    (12, 40_001, 1, 1), (13, 40_001, 1, 1),                              # 64 and 32 lanes
    (32, 2_047, 0, 0), (130, 4_095, 1, 1), (4_097, 63, 1, 0), (999, 5_119, 0, 1),       # 8 lanes, 1 to 8 waves
    (32, 1_003, 1, 1), (64, 20_005, 1, 0), (65, 9_001, 1, 1), (161, 9_001, 1, 0), (256, 2_055, 1, 1),     # one wave, 32 to 8 lanes
    (515, 20_480, 1, 1), (1_025, 10_241, 0, 0), (513, 20_481, 1, 0),     # 160 tiles of 16 lanes and one more or less
    (64, 40_959, 0, 0), (300, 140_001, 1, 1), (700, 61_441, 0, 1),       # 32 lanes
    (20, 1_200_001, 0, 0), (64, 262_143, 0, 1), (127, 41_000, 0, 0),     # 64 lanes
    (300, 900_003, 0, 0), (700, 720_005, 1, 1), (300, 900_032, 0, 0),    # beyond 1 GB
    (2_900, 320_001, 1, 1), (700, 412_000, 1, 0), (700, 394_240, 1, 0),  # more than half a GB: 2 waves of 64 lanes or 1 of 32
    (90, 2_900_001, 0, 1), (40, 7_100_001, 1, 0), (4_096, 33_281, 0, 0),
    (300, 335_001, 0, 1), (699, 290_001, 1, 1), (1_024, 97_900, 0, 1), (2_048, 49_003, 0, 1),    # off the lines beyond 350 MB: 64 and 32 lanes
    (699, 20_003, 0, 0), (700, 20_003, 0, 0),                            # from the first row to the last and the other way
    (3, 8_300_003, 0, 1),                                                # tiles widened so that there are not too many
])
def test_against_binary64(N, P, dtype, odd):
    torch.manual_seed(N + P)
    stride = P + 3 if odd else (P + 63) // 64 * 64                       # rows off and on the cache lines
    X = torch.randn(N, stride, device=DEV, dtype=torch.float32)
    X += torch.randn(N, 1, device=DEV)
    X = X.to(torch.float32 if dtype == 0 else torch.bfloat16)[:, odd:P + odd]
    out = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
    print(f"distortion N={N} P={P} dtype={dtype} odd={odd}", flush=True)
    binding.dist_to_mean_static(X, out)
    want = torch.zeros((), dtype=torch.float64, device=DEV)
    scale = torch.zeros((), dtype=torch.float64, device=DEV)
    width = max(1, (1 << 25) // N)
    for a in range(0, P, width):
        Y = X[:, a:a + width].double()
        want += ((Y - Y.mean(0, keepdim=True)) ** 2).sum() / N
        scale += ((Y - Y[:1]) ** 2).sum() / N
    # s2 and s1 are sums of N terms in binary64, of differences from row 0, and s1^2 / N <= s2
    bound = 4.0 * (N + 64) * 2.0 ** -53 * float(scale)
    assert abs(float(out) - float(want)) <= bound, (float(out), float(want), bound)
