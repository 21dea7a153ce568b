"""Plans of whole-grid passes (csrc/grid_plan.h), compiled for the host: over all the shapes that have
one, what the two kernels take for granted.  No GPU needed."""
import shutil
import subprocess

import pytest

import __graft_entry__ as entry

# Every plan of a sweep over grids, row lengths, strides, alignments and what a run may ask for.
SWEEP = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "grid_plan.h"
using namespace moshpit;

static int bad = 0;
static void say(const char *what, const GridPlan &p, int dtype, const GridAsk &a)
{
    if (++bad <= 20)
        std::printf("%s: M=%d d=%d dtype=%d row %lld of %lld bytes, absent=%d refresh=%d distortions=%d rounds=%d: tile %d x %d parts, "
                    "%d threads, means %d bits %d\n", what, p.M, p.d, dtype, (long long)p.valid_bytes, (long long)p.row_bytes, a.absent,
                    a.refresh, a.distortions, a.rounds, p.Wb, p.phases, p.threads, p.means, p.bits);
}

static void check(const GridPlan &p, int dtype, const GridAsk &a);

int main()
{
    long plans = 0;
    for (int32_t M = 2; M <= 32; ++M) {
        int32_t d = 1;
        for (int64_t N = M; N <= kGridMaxPeers; N *= M, ++d)
            for (int dtype = 0; dtype < 2; ++dtype) {
                const int64_t es = dtype == 0 ? 4 : 2, line = 128 / es;
                std::vector<int64_t> lengths;
                for (double x = 16.0 / es; x * es * N < 20e9; x *= 1.7)
                    for (int64_t n : {int64_t(x), int64_t(x) / line * line + line, int64_t(x) | 1}) lengths.push_back(n);
                for (int64_t P : lengths) {
                    std::vector<int64_t> strides = {P, (P + line - 1) / line * line};
                    for (double bytes : {34e6, 300e6})
                        if (bytes > double(N) * P * es) strides.push_back(int64_t(bytes / (N * es)) / line * line + line);
                    for (int64_t stride : strides)
                        for (int ask = 0; ask < 16; ++ask)
                            for (int32_t rounds : {0, 1, 2, 4, 5, 9, 70}) {
                                GridAsk a;
                                a.absent = ask & 1;
                                a.refresh = a.absent && (ask & 2);
                                a.distortions = ask & 4;
                                a.local_step = ask & 8;
                                a.rounds = rounds;
                                GridPlan p;
                                for (uintptr_t at : {uintptr_t(4096), uintptr_t(4096 + es)})
                                    if (plan_grid(dtype, N, M, d, P, stride, reinterpret_cast<void *>(at), 1, a, &p)) {
                                        check(p, dtype, a);
                                        ++plans;
                                    }
                            }
                }
            }
    }
    std::printf("%ld plans\n", plans);
    return bad != 0 || plans < 100000;
}
"""


def run_host(tmp_path, source, text=""):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "plan.cpp"
    src.write_text(source)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", entry.CSRC, str(src), "-o",
                           str(tmp_path / "plan")])
    return subprocess.run([str(tmp_path / "plan")], input=text, capture_output=True, text=True, timeout=120)


FITS = SWEEP + r"""
static void check(const GridPlan &p, int dtype, const GridAsk &a)
{
    const int64_t part = p.Wb / p.phases, es = dtype == 0 ? 4 : 2;
    if (p.threads % 64 != 0 || p.threads > (p.phases == 1 ? 1024 : 512) || p.max_rounds < 1 || p.max_rounds > 64) say("threads or rounds", p, dtype, a);
    // a thread's slots hold the tile, and every column is in some tile
    if (static_cast<int64_t>(p.threads) * 16 * kPhaseSlots < p.N * part || p.tiles * p.Wb < p.valid_bytes) say("tile", p, dtype, a);
    if (!p.means) return;
    if (a.local_step) say("local step", p, dtype, a);
    // LDS of a pass of max_rounds rounds with distortions
    const int64_t waves = p.threads / 64, sums = a.distortions ? (waves * (part / es) + p.dist_window * waves) * 8 : 0;
    if (p.red_offset + sums > kLdsPerBlock || p.red_offset % 8 != 0 || p.zero_at + part > kLdsPerBlock) say("LDS", p, dtype, a);
    if (!a.absent) return;
    // tables: a place has 13 bits, a lane one item of 8 positions, a register a round's words
    if (p.zero_at / 16 >= 1 << 13 || p.M != 8 * p.split || static_cast<int64_t>(p.groups) * (part / 16) * p.split > p.threads) say("places", p, dtype, a);
    if (2 << p.words_shift != p.N || (part >= kLeastLdsPart && p.threads >> p.words_shift < 1)) say("words", p, dtype, a);
    if (p.bits && (p.M != 16 || part != 16 || p.threads != 2 * p.groups || a.refresh || a.distortions)) say("bits", p, dtype, a);
}
"""


def test_every_plan_fits_its_kernel(tmp_path):
    """Threads, LDS and tables of every plan are what the kernels assume."""
    out = run_host(tmp_path, FITS)
    assert out.returncode == 0, out.stdout


ROUNDS = SWEEP + r"""
static void check(const GridPlan &p, int dtype, const GridAsk &a)
{
    if (!p.means) return;
    GridAsk other = a;
    other.local_step = true;                 // (takes the kernel with M copies of a mean)
    GridPlan q;
    const int64_t es = dtype == 0 ? 4 : 2;
    if (!plan_grid(dtype, p.N, p.M, p.d, p.valid_bytes / es, p.row_bytes / es, reinterpret_cast<void *>(4096), 1, other, &q)) return;
    // (measured ahead all the same: see sums_leave_in_between)
    if (p.max_rounds < q.max_rounds && p.max_rounds < (p.M == 6 && p.N == 216 ? 10 : 24)) say("fewer rounds a pass", p, dtype, a);
}
"""


def test_one_mean_per_group_takes_no_more_passes(tmp_path):
    """A run does not read and write the state more often because the kernel with one mean per group takes it,
    but for runs of more than 24 rounds (6 x 6 x 6: 10)."""
    out = run_host(tmp_path, ROUNDS)
    assert out.returncode == 0, out.stdout
