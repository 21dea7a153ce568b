"""Sizes and choices of multi-round passes (csrc/pass_rules.h), compiled for the host and checked
over the shapes they serve.  No GPU needed."""
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


def run_host(tmp_path, source):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "rules.cpp"
    src.write_text(source)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", entry.CSRC, str(src), "-o",
                           str(tmp_path / "rules")])
    return subprocess.run([str(tmp_path / "rules")], capture_output=True, text=True, timeout=120)


def test_tables_of_a_long_run_are_bounded_and_hold_whole_passes(tmp_path):
    """Whatever the grid, the tables take at most 16 MiB (or one pass), their indexes stay below
    2^31 and the launch that fills them below 2^32 threads; the distortion sums take at most 256 MiB
    (or one round)."""
    out = run_host(tmp_path, SOURCE)
    assert out.returncode == 0, out.stdout
