"""Sizes and choices of multi-round passes (csrc/pass_rules.h), compiled for the host and checked
over the shapes they serve and against measured times.  No GPU needed."""
import os
import shutil
import subprocess

import pytest

import __graft_entry__ as entry

SOURCE = r"""
#include <cstdio>
#include "pass_rules.h"
using namespace moshpit;
int main()
{
    int bad = 0;
    for (int64_t M = 2; M <= 32; ++M)
        for (int64_t N = M; N <= 4096; N *= M)
            for (int refresh = 0; refresh <= 1; ++refresh)
                for (int64_t most = 1; most <= 64; most += most < 16 ? 1 : 12) {
                    const int64_t n = grid_table_rounds(N, static_cast<int32_t>(M), refresh != 0, most);
                    const int64_t bytes = n * grid_table_round_bytes(N, static_cast<int32_t>(M), refresh != 0);
                    const bool whole_passes = n >= most && n % most == 0;
                    const bool bounded = bytes <= kGridTableBytes || n == most;
                    const bool small = n * (N / M) < (int64_t(1) << 31) && (n + N / 1024 + 1) * 1024 < (int64_t(1) << 32);
                    if (!whole_passes || !bounded || !small) {
                        std::printf("M=%lld N=%lld refresh=%d most=%lld: %lld rounds, %lld bytes\n", (long long)M, (long long)N,
                                    refresh, (long long)most, (long long)n, (long long)bytes);
                        ++bad;
                    }
                }
    // a pass with distortions: at least one round, and either its sums fit the buffer or it is one round
    for (int64_t tiles = 1; tiles < (int64_t(1) << 31); tiles *= 3)
        for (int most = 4; most <= 64; most += 12) {
            const int n = grid_pass_rounds(most, tiles);
            const bool fits = (n + 1) * tiles * 8 <= kGridPartialBytes;
            if (n < 1 || n > most || (!fits && n != 1) || (fits && n < most && (n + 2) * tiles * 8 <= kGridPartialBytes)) {
                std::printf("tiles=%lld most=%d: %d rounds\n", (long long)tiles, most, n);
                ++bad;
            }
        }
    return bad;
}
"""


def run_host(tmp_path, source, text=""):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "rules.cpp"
    src.write_text(source)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", entry.CSRC, str(src), "-o",
                           str(tmp_path / "rules")])
    return subprocess.run([str(tmp_path / "rules")], input=text, capture_output=True, text=True, timeout=120)


def test_tables_of_a_long_run_are_bounded_and_hold_whole_passes(tmp_path):
    """Whatever the grid, the tables take at most 16 MiB (or one pass), their indexes stay below
    2^31 and the launch that fills them below 2^32 threads; the distortion sums take at most 256 MiB
    (or one round)."""
    out = run_host(tmp_path, SOURCE)
    assert out.returncode == 0, out.stdout


# Measured on MI355X: grid, rounds, fraction of the peers absent, group-skip, fused passes of the other way
# (rounds, whole grid, blocks per compute unit), tile of the whole-grid pass (bytes of a row, parts, threads,
# LDS bytes, rounds), curve; microseconds of the other way and of the pass with M copies of a mean (some of the longer runs
# take the kernel with one mean per group by now: test_grid_plan.py has measured runs of that one).
MEASURED = [
    (16, 2, 4, 1_048_576, 2, 0.0, 0, [], (256, 1, 512, 65_800, 64), 0, 733, 408),
    (16, 2, 4, 1_048_576, 2, 0.2, 0, [], (256, 1, 512, 65_800, 64), 0, 597, 402),
    (16, 2, 4, 1_048_576, 2, 0.9, 0, [], (256, 1, 512, 65_800, 64), 0, 166, 260),
    (16, 2, 4, 1_048_576, 8, 0.9, 0, [], (256, 1, 512, 65_800, 64), 0, 903, 459),
    (16, 2, 4, 1_048_576, 10, 0.05, 0, [(10, 1, 2)], (256, 1, 512, 65_800, 64), 1, 1041, 818),
    (32, 2, 4, 4_194_304, 2, 0.0, 0, [], (128, 2, 512, 66_560, 64), 0, 11_100, 7_811),
    (32, 2, 4, 4_194_304, 2, 0.9, 0, [], (128, 2, 512, 66_560, 64), 0, 3_212, 5_766),
    (32, 2, 4, 4_194_304, 8, 0.2, 0, [], (128, 2, 512, 66_560, 64), 0, 36_602, 9_485),
    (32, 2, 4, 4_194_304, 8, 0.2, 0, [(8, 1, 1)], (128, 2, 512, 66_560, 64), 0, 10_602, 9_302),
    (32, 2, 4, 4_194_304, 8, 0.2, 1, [], (128, 2, 512, 66_560, 64), 0, 2_475, 5_100),
    (32, 2, 4, 4_194_304, 8, 0.05, 1, [], (128, 2, 512, 66_560, 64), 0, 11_723, 8_317),
    (16, 3, 2, 262_144, 2, 0.2, 0, [], (32, 2, 512, 73_728, 14), 0, 1_151, 1_654),
    (16, 3, 2, 262_144, 2, 0.2, 0, [(2, 0, 2)], (32, 2, 512, 73_728, 14), 0, 864, 1_630),
    (16, 3, 2, 262_144, 8, 0.2, 0, [(2, 0, 2)] * 4, (32, 2, 512, 73_728, 14), 0, 3_600, 2_174),
    (16, 3, 2, 262_144, 8, 0.2, 1, [], (32, 2, 512, 73_728, 14), 0, 597, 1_325),
    (3, 7, 4, 131_072, 8, 0.2, 0, [(4, 0, 2), (4, 0, 2)], (32, 1, 576, 72_171, 6), 0, 1_172, 2_006),
    (7, 4, 2, 131_072, 2, 0.2, 0, [], (32, 2, 320, 40_817, 44), 0, 360, 622),
    (7, 4, 2, 131_072, 8, 0.0, 0, [], (32, 2, 320, 40_817, 44), 0, 1_660, 1_064),
    (4, 2, 4, 65_536, 2, 0.0, 0, [], (256, 1, 64, 4_112, 64), 0, 7.9, 6.0),
]

CHOICE = r"""
#include <cmath>
#include <cstdio>
#include <vector>
#include "pass_rules.h"
using namespace moshpit;
int main()
{
    int M, d, es, rounds, skip, n, row, parts, threads, lds, most, curve;
    long long P;
    double absent, other_us, pass_us;
    int bad = 0;
    while (std::scanf("%d %d %d %lld %d %lf %d %d", &M, &d, &es, &P, &rounds, &absent, &skip, &n) == 8) {
        RunSize z;
        z.M = M;
        z.element_bytes = es;
        z.N = 1;
        for (int q = 0; q < d; ++q) z.N *= M;
        z.valid_bytes = z.row_bytes = P * es;
        const Participation w = absent > 0.0 ? independent_presence(1.0 - absent, M, skip != 0) : Participation{};
        double other = 0.0;
        int distortions = 1;
        for (int k = 0; k < n; ++k, ++distortions) {
            int r, whole, blocks;
            if (std::scanf("%d %d %d", &r, &whole, &blocks) != 3) return 99;
            other += fused_pass_us(z, w, r, whole != 0, blocks);
        }
        if (n == 0) {
            other = rounds * single_round_us(z, w);
            distortions += rounds;
        }
        if (std::scanf("%d %d %d %d %d %d %lf %lf", &row, &parts, &threads, &lds, &most, &curve, &other_us, &pass_us) != 8) return 99;
        GridTiles t;
        t.row_bytes = row;
        t.parts = parts;
        t.threads = threads;
        t.lds_bytes = lds;
        t.max_rounds = most;
        t.tiles = (z.valid_bytes + row - 1) / row;
        if (curve) other += distortions * distortion_us(z);
        const double pass = grid_passes_us(z, w, t, rounds, curve ? distortions : 0);
        if ((kRoundsAhead * pass <= other) != (pass_us < other_us)) {
            std::printf("%d^%d x %lld, %d rounds, %.2f absent: other way %.0f (measured %.0f), pass %.0f (%.0f)\n", M, d, P, rounds,
                        absent, other, other_us, pass, pass_us);
            ++bad;
        }
    }
    // masks looked at one by one: as drawn, nobody, everybody, and one group of each round only
    for (int kind = 0; kind < 4; ++kind)
        for (int group_skip = 0; group_skip <= 1; ++group_skip) {
            const int64_t N = 4096, R = 12, t0 = 5;
            std::vector<uint8_t> masks(N * R);
            uint32_t x = 12345;
            for (int64_t r = 0; r < R; ++r)
                for (int64_t i = 0; i < N; ++i) {
                    x = x * 1664525u + 1013904223u;
                    int64_t S = 1;
                    for (int64_t q = 0; q < (t0 + r) % 3; ++q) S *= 16;
                    const bool first_group = i % S == 0 && i / (S * 16) == 0;
                    masks[r * N + i] = kind == 0 ? (x >> 16) % 10 < 7 : kind == 1 ? 0 : kind == 2 ? 255 : first_group;
                }
            const Participation got = sampled_presence(masks.data(), R, N, 16, 3, t0, group_skip != 0);
            const Participation want = independent_presence(kind == 0 ? 0.7 : kind == 2 ? 1.0 : 0.0, 16, group_skip != 0);
            // (2,000 draws; the last kind: one group of 256, and 64 peers looked at)
            const double room = kind == 3 ? 0.1 : 0.06;
            if (std::fabs(got.present - want.present) > room || std::fabs(got.averaged - want.averaged) > room ||
                std::fabs(got.groups - want.groups) > room || std::fabs(got.ever(R) - want.ever(R)) > room) {
                std::printf("masks %d, group-skip %d: present %.3f averaged %.3f groups %.3f ever %.3f\n", kind, group_skip, got.present,
                            got.averaged, got.groups, got.ever(R));
                ++bad;
            }
        }
    return bad;
}
"""


def test_the_cheaper_way_of_measured_runs_is_taken(tmp_path):
    """Whole-grid pass or the other way: the prices put runs whose ways were measured at least 12 %
    apart in the right order, and the masks of a caller are estimated as they are."""
    text = ""
    for M, d, es, P, rounds, absent, skip, fused, tile, curve, other, whole in MEASURED:
        assert max(other, whole) > 1.12 * min(other, whole)
        text += " ".join(map(str, (M, d, es, P, rounds, absent, skip, len(fused), *(x for f in fused for x in f), *tile, curve,
                                   other, whole))) + "\n"
    out = run_host(tmp_path, CHOICE, text)
    assert out.returncode == 0, out.stdout
