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
    // LDS of a pass
    int32_t sums_at = 0;
    const int64_t lds = p.means ? means_lds_bytes(p, a.absent, p.max_rounds, a.distortions, es, &sums_at)
                                : copies_lds_bytes(p, p.max_rounds, a.distortions, es, &sums_at);
    if (lds > kLdsPerBlock || sums_at % 8 != 0 || (p.means && (sums_at != p.red_offset || p.zero_at + part > p.rcp_at))) say("LDS", p, dtype, a);
    if (!p.means) return;
    if (a.local_step) say("local step", p, dtype, a);
    // the waves that share a distortion: half of the block's, or one less where that holds the sums of 24 rounds
    const int32_t waves = p.threads / 64, half = waves > 1 ? waves / 2 : 1;
    if (a.distortions && p.sharers != half && (p.sharers != half - 1 || p.sharers < 1 || p.max_rounds < 24)) say("sharers", p, dtype, a);
    if (!a.absent) return;
    // tables: a place has 13 bits, a lane one item of 8 positions, a register a round's words
    if (p.zero_at / 16 >= 1 << 13 || p.M != 8 * p.split || static_cast<int64_t>(p.groups) * (part / 16) * p.split > p.threads) say("places", p, dtype, a);
    if (2 << p.words_shift != p.N || (part >= kLeastLdsPart && p.threads >> p.words_shift < 1)) say("words", p, dtype, a);
    if (a.distortions && part >= kLeastLdsPart && 128 * p.sharers != p.threads) say("halves", p, dtype, a);
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
    // (those with distortions, 6 x 6 x 6 in bfloat16 least)
    if (p.max_rounds < q.max_rounds && p.max_rounds < (p.M == 6 && p.N == 216 ? 10 : 24)) say("fewer rounds a pass", p, dtype, a);
}
"""


def test_one_mean_per_group_takes_no_more_passes(tmp_path):
    """A run does not read and write the state more often because the kernel with one mean per group takes it,
    but for runs of more than 24 rounds (6 x 6 x 6: 10)."""
    out = run_host(tmp_path, ROUNDS)
    assert out.returncode == 0, out.stdout


KERNELS = SWEEP.replace("return bad != 0", "built(); return bad != 0").replace("int main()", "static void built();\nint main()") + r"""
#include <set>
#include <tuple>
static std::set<std::tuple<int, int, int, int, int, int>> asked;
static void check(const GridPlan &p, int dtype, const GridAsk &a)
{
    if (!p.means) return;
    for (int dist = 0; dist <= (a.distortions ? 1 : 0); ++dist) {       // (a pass none of whose distortions is returned does without)
        const MeanKernel k = mean_kernel(p, a.absent, dist != 0);
        if (!mean_kernel_built(dtype, k.split, k.half, k.nt, k.dist, k.tab)) say("no such kernel", p, dtype, a);
        asked.insert({dtype, k.split, k.half, k.nt, k.dist, k.tab});
    }
}
static void built()
{
    int n = 0;
    for (int dtype : {0, 1})
        for (int split : {1, 2, 4})
            for (int half : {0, 1, 2, 32})
                for (int nt : {0, 1})
                    for (int dist : {0, 1})
                        for (int tab : {kClosed, kLds, kAheadOnly, kBits}) {
                            if (!mean_kernel_built(dtype, split, half, nt != 0, dist != 0, tab)) continue;
                            ++n;
                            if (asked.count({dtype, split, half, nt, dist, tab}) == 0) {
                                std::printf("never asked for: dtype %d split %d half %d nt %d dist %d tab %d\n", dtype, split, half, nt, dist, tab);
                                ++bad;
                            }
                        }
    std::printf("%d kernels\n", n);
}
"""


def test_the_kernels_that_are_built_are_those_that_plans_ask_for(tmp_path):
    out = run_host(tmp_path, KERNELS)
    assert out.returncode == 0, out.stdout


TABLES = SWEEP.replace('#include "grid_plan.h"', '#include "pass_rules.h"') + r"""
static void check(const GridPlan &p, int dtype, const GridAsk &a)
{
    if (!p.means || !a.absent) return;
    const int64_t pass_most = grid_pass_rounds(p.max_rounds, a.distortions ? p.tiles * p.phases : 0);
    const int64_t most = table_rounds(mean_table_round_bytes(p.N, p.M, p.split), pass_most);
    if (most < pass_most || most % pass_most != 0 || (p.bits && pass_most % 16 != 0)) say("passes", p, dtype, a);
    for (int skip = 0; skip <= 1; ++skip) {
        const MeanTableWords full = mean_table_words(p, most, pass_most, a.distortions, skip != 0);
        // (final places: 2 bytes for every slot of a pass)
        const int64_t places = 2 * mean_place_stride(p) * (most / pass_most);
        if (4 * full.total > kGridTableBytes + places && most > pass_most) say("bound", p, dtype, a);
        for (int64_t rounds : {int64_t(1), int64_t(5), int64_t(17), pass_most, pass_most + 1, most - 1, most}) {
            if (rounds < 1 || rounds > most) continue;
            const MeanTableWords w = mean_table_words(p, rounds, pass_most, a.distortions, skip != 0);
            if (w.total > full.total || w.total >= (int64_t(1) << 31)) say("size", p, dtype, a);
            if (w.entries % 4 != 0 || w.move_rows % 4 != 0 || w.move_bytes % 4 != 0 || w.places % 4 != 0) say("alignment", p, dtype, a);
            // what the kernels index: the last word of each piece lies before the next
            const int64_t width = p.bits ? 1 : 4 * p.split, last = rounds - 1;
            if ((last * p.groups + p.groups - 1) * width + width > w.move_rows - w.entries) say("entries", p, dtype, a);
            if (p.bits && (last / 2 * p.threads + p.threads - 1 >= w.move_bytes - w.move_rows ||
                           last / 4 * p.threads + p.threads - 1 >= w.places - w.move_bytes)) say("rows", p, dtype, a);
            if (p.bits && (last / 16 * 8 + 8) * p.threads > w.move_bytes - w.move_rows) say("rows read ahead", p, dtype, a);
            if (2 * (w.moves - w.places) < (last / pass_most + 1) * mean_place_stride(p)) say("places", p, dtype, a);
            if (w.terms - w.moves < rounds * p.N || w.move_counts - w.terms < (a.distortions ? rounds * (p.N + p.groups) : 0)) say("moves", p, dtype, a);
            if (w.term_counts - w.move_counts < rounds || w.bitmaps - w.term_counts < rounds || w.total - w.bitmaps < skip * rounds * p.groups) say("counts", p, dtype, a);
        }
    }
}
"""


def test_tables_of_one_mean_per_group_are_bounded_and_do_not_overlap(tmp_path):
    out = run_host(tmp_path, TABLES)
    assert out.returncode == 0, out.stdout


CHOICE = r"""
#include <cstdio>
#include "pass_rules.h"
using namespace moshpit;
int main()
{
    int M, d, dtype, rounds, absent, skip, curve, refresh;
    double mb;
    while (std::scanf("%d %d %d %lf %d %d %d %d %d", &M, &d, &dtype, &mb, &rounds, &absent, &skip, &curve, &refresh) == 9) {
        const int64_t es = dtype == 0 ? 4 : 2;
        int64_t N = 1;
        for (int q = 0; q < d; ++q) N *= M;
        const int64_t P = static_cast<int64_t>(mb * 1e6) / (N * es) / 8 * 8;
        GridAsk a;
        a.absent = absent != 0;
        a.distortions = curve != 0;
        a.refresh = refresh != 0;
        a.rounds = rounds;
        // (a peer that is refreshed was away for two rounds)
        const double q = refresh ? (1.0 - 0.01 * absent) / (1.0 + 0.01 * absent) : 1.0 - 0.01 * absent;
        const Participation who = absent ? independent_presence(q, M, skip != 0) : Participation{};
        a.averaged = who.averaged;
        a.live = who.groups;
        GridPlan p;
        // (means, blocks of a pass that share a compute unit)
        int32_t at = 0;
        const bool planned = plan_grid(dtype, N, M, d, P, P, reinterpret_cast<void *>(4096), 0, a, &p);
        const int64_t lds = p.means ? means_lds_bytes(p, a.absent, rounds, a.distortions, es, &at) : copies_lds_bytes(p, rounds, a.distortions, es, &at);
        // (and are passes cheaper than rounds one by one?)
        RunSize z;
        z.N = N;
        z.M = M;
        z.element_bytes = static_cast<int32_t>(es);
        z.valid_bytes = z.row_bytes = P * es;
        const GridTiles t = grid_tiles(p, a, es);
        const double by_rounds = rounds * single_round_us(z, who) + (refresh ? (rounds - 1) * refresh_us(z) : 0.0) + (curve ? (rounds + 1) * distortion_us(z) : 0.0);
        const bool passes = planned && !rounds_ahead(by_rounds, grid_passes_us(z, who, t, rounds, curve ? rounds + 1 : 0), t);
        std::printf("%d %d %d %d\n", planned ? p.means : -1, static_cast<int>(blocks_by_lds(lds)), passes, p.means ? t.lds_bytes == lds : 1);
    }
}
"""

# Measured on MI355X: grid, type, MB, rounds, % absent, group-skip, curve, refresh; microseconds with M copies of a mean and
# with one mean per group.
MEASURED = [
    # as many blocks as tiles at once, or two turns
    (7, 3, 0, 20, 4, 0, 0, 0, 0, 15.8, 13.7), (7, 3, 0, 28, 4, 0, 0, 0, 0, 19.1, 22.4), (7, 3, 0, 28, 20, 0, 0, 0, 0, 47.9, 53.0),
    (7, 3, 1, 28, 20, 0, 0, 0, 0, 63.3, 69.6), (7, 3, 0, 36, 10, 0, 0, 0, 0, 41.6, 36.6), (8, 2, 0, 24, 4, 0, 0, 0, 0, 13.7, 12.2),
    (8, 2, 0, 33, 4, 0, 0, 0, 0, 16.4, 19.1), (8, 2, 0, 33, 64, 0, 0, 0, 0, 120.6, 85.4), (8, 2, 0, 40, 6, 0, 0, 0, 0, 23.6, 22.0),
    (24, 2, 0, 30, 10, 0, 0, 0, 0, 32.1, 33.9), (24, 2, 0, 30, 32, 0, 0, 0, 0, 94.9, 75.9), (5, 3, 0, 36, 4, 0, 0, 0, 0, 20.2, 21.8),
    (5, 3, 0, 28, 4, 0, 0, 0, 0, 18.5, 15.0), (8, 3, 0, 28, 6, 0, 0, 0, 0, 18.6, 20.9), (9, 2, 0, 33, 4, 0, 0, 0, 0, 24.2, 20.2),
    (8, 3, 0, 28, 1, 0, 0, 1, 0, 40.1, 43.7), (8, 3, 0, 28, 5, 0, 0, 1, 0, 56.5, 53.8), (8, 3, 1, 28, 4, 0, 0, 0, 0, 25.2, 23.2),
    (24, 2, 1, 33, 8, 0, 0, 0, 0, 39.7, 36.5), (9, 2, 1, 30, 2, 0, 0, 1, 0, 68.7, 52.6), (8, 3, 1, 32, 32, 0, 0, 0, 0, 112.4, 82.5),
    # small states with failures
    (16, 3, 0, 33, 5, 10, 0, 0, 0, 55.3, 60.2), (16, 3, 1, 40, 8, 10, 0, 0, 0, 63.4, 66.5), (32, 2, 0, 36, 5, 10, 0, 0, 0, 28.1, 30.8),
    (8, 3, 0, 33, 5, 10, 0, 0, 0, 38.4, 40.9), (8, 3, 0, 44, 8, 10, 0, 0, 0, 40.1, 35.9), (16, 2, 0, 36, 5, 10, 0, 0, 0, 25.1, 23.7),
    (8, 3, 0, 200, 5, 10, 0, 0, 1, 108.9, 86.5), (32, 2, 0, 40, 10, 10, 0, 1, 0, 106.2, 92.1), (16, 3, 0, 200, 5, 10, 0, 1, 0, 249, 209),
    # two column parts in place of one
    (8, 3, 0, 1000, 4, 0, 0, 0, 0, 420, 443), (8, 3, 0, 1000, 8, 0, 0, 0, 0, 502, 425), (8, 3, 0, 1000, 5, 10, 0, 0, 0, 433, 457),
    (8, 3, 0, 1000, 8, 10, 0, 0, 0, 515, 446), (8, 3, 0, 1000, 5, 10, 0, 1, 0, 867, 1204), (8, 3, 0, 3000, 20, 10, 0, 1, 0, 7080, 8215), (8, 3, 0, 3000, 64, 10, 0, 1, 0, 21464, 20267),
    (8, 3, 0, 1000, 5, 10, 0, 0, 1, 554, 458), (8, 3, 0, 200, 5, 10, 0, 1, 0, 198.7, 170.4), (8, 3, 0, 1000, 5, 0, 0, 1, 0, 838, 660),
    (13, 3, 0, 1000, 5, 0, 0, 1, 0, 1244, 959), (13, 3, 0, 1000, 12, 0, 0, 1, 0, 2196, 1313), (13, 3, 0, 1000, 4, 0, 0, 0, 0, 776, 600),
    (13, 3, 1, 1000, 2, 0, 0, 1, 0, 1586, 1143), (24, 2, 0, 1000, 5, 0, 0, 1, 0, 1127, 1078), (24, 2, 0, 1000, 40, 0, 0, 1, 0, 6600, 4579), (24, 2, 0, 3000, 12, 0, 0, 1, 0, 6032, 4989),
    (24, 2, 0, 1000, 4, 0, 0, 0, 0, 532, 497), (32, 2, 0, 250, 4, 0, 0, 0, 0, 99, 108), (24, 2, 1, 1000, 8, 0, 0, 0, 0, 3055, 828),
    # who is absent (60 MB and more, 12 rounds unless stated): curves, refresh, groups without an average, half of the peers
    (16, 2, 0, 300, 12, 30, 0, 1, 0, 521, 365), (16, 2, 0, 300, 12, 80, 0, 1, 0, 515, 527), (32, 2, 0, 1500, 12, 90, 0, 1, 0, 2530, 3692),
    (8, 3, 0, 60, 12, 70, 0, 1, 0, 145, 198), (16, 3, 0, 300, 12, 90, 0, 1, 0, 602, 758),
    (8, 3, 1, 300, 12, 95, 0, 0, 1, 178, 204), (16, 2, 0, 300, 12, 95, 0, 0, 1, 143, 125),
    (8, 3, 1, 1500, 12, 95, 0, 0, 0, 845, 1184), (8, 3, 1, 300, 12, 80, 0, 0, 0, 306, 293), (8, 3, 0, 300, 12, 90, 0, 0, 0, 170, 193),
    (16, 2, 0, 300, 12, 30, 1, 0, 0, 94, 117), (32, 2, 1, 1500, 12, 10, 1, 0, 0, 746, 822), (32, 2, 1, 1500, 12, 95, 0, 0, 0, 1253, 1048),
    (8, 3, 0, 300, 12, 50, 0, 0, 0, 212, 233), (16, 3, 0, 60, 12, 70, 0, 0, 0, 84, 94), (16, 3, 1, 300, 12, 50, 0, 0, 0, 346, 394),
    (16, 3, 1, 300, 6, 50, 0, 0, 0, 311, 277),
    # curves: two parts with a mean per group; few rounds, many absent
    (24, 2, 0, 438.8, 2, 0, 0, 1, 0, 320, 365), (16, 2, 0, 205.5, 24, 50, 0, 1, 0, 674, 549),
    (16, 2, 0, 80.4, 12, 50, 0, 1, 0, 163, 185.8), (32, 2, 0, 58, 12, 30, 0, 1, 0, 144.7, 126.9),
    (16, 3, 0, 182.4, 5, 70, 0, 1, 0, 238, 266), (16, 3, 0, 55, 24, 60, 0, 1, 0, 311, 266),
    (16, 3, 1, 184.1, 5, 95, 0, 1, 0, 329, 360), (16, 3, 1, 191.1, 8, 50, 0, 1, 0, 469, 419),
    (8, 3, 0, 219.5, 8, 50, 0, 1, 0, 298, 323),
    # curves with returning peers
    (8, 3, 0, 80.2, 12, 50, 0, 1, 1, 203, 248), (16, 2, 0, 79.9, 5, 50, 0, 1, 1, 111, 126.4),
    (16, 2, 0, 217.4, 8, 50, 0, 1, 1, 326, 281), (32, 2, 0, 470.5, 8, 60, 0, 1, 1, 791, 897),
    (16, 3, 0, 187.3, 24, 20, 0, 1, 1, 928, 590), (16, 3, 0, 376.9, 8, 90, 0, 1, 1, 665, 764),
]


def plans(tmp_path, rows):
    """(one mean per group, blocks per compute unit, passes instead of rounds, LDS as priced) of each."""
    out = run_host(tmp_path, CHOICE, "".join(" ".join(map(str, row)) + "\n" for row in rows))
    assert out.returncode == 0
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def test_the_faster_kernel_of_measured_runs_is_taken(tmp_path):
    got = plans(tmp_path, [row[:9] for row in MEASURED])
    wrong = [(row, means) for row, (means, *_) in zip(MEASURED, got, strict=True) if means != (row[10] < row[9])]
    assert not wrong, wrong


def test_odd_numbers_of_waves_share_a_compute_unit_as_often(tmp_path):
    """Curves whose blocks have 1, 5, 7 or 9 waves: next to the distortions' sums there is room for as many blocks as before two rounds'
    sums were kept, and for one column part."""
    rows = [(12, 2, 1, 300, 24, 0, 0, 1, 0), (12, 2, 1, 1000, 64, 0, 0, 1, 0), (13, 3, 0, 9, 4, 0, 0, 1, 0), (13, 3, 0, 1000, 10, 0, 0, 1, 0),
            (20, 2, 0, 300, 30, 0, 0, 1, 0), (24, 2, 0, 300, 30, 0, 0, 1, 0), (23, 2, 1, 300, 30, 0, 0, 1, 0), (5, 3, 0, 9, 10, 0, 0, 1, 0)]
    assert [g[:2] for g in plans(tmp_path, rows)] == [(1, 3), (1, 3), (1, 4), (1, 2), (1, 2), (1, 3), (1, 2), (1, 14)]


def test_256_peers_with_failures_fit_a_compute_unit_four_times(tmp_path):
    """In tiles of 128 bytes, as with M copies of a mean."""
    assert plans(tmp_path, [(16, 2, dtype, mb, 16, 10, 0, 0, 0) for dtype in (0, 1) for mb in (33, 100)]) == [(1, 4, 1, 1)] * 4


# The same columns; microseconds round by round and in passes with one mean per group.
WAYS = [
    (16, 2, 1, 1646, 6, 95, 0, 0, 0, 322, 522), (16, 2, 1, 494, 6, 95, 0, 0, 0, 110, 173), (16, 2, 1, 513, 8, 95, 0, 0, 0, 156, 214),
    (16, 3, 1, 370, 8, 90, 0, 0, 0, 212, 293), (16, 3, 1, 487, 16, 95, 0, 0, 0, 387, 595), (16, 3, 0, 804, 5, 90, 0, 0, 0, 296, 424),
    (32, 2, 1, 304, 6, 95, 0, 0, 0, 110, 149), (16, 2, 0, 735, 12, 95, 0, 0, 0, 412, 304), (16, 2, 1, 307, 6, 90, 0, 0, 0, 177, 133),
    (32, 2, 0, 105, 16, 90, 0, 0, 0, 148, 95), (32, 2, 1, 835, 10, 95, 0, 0, 0, 730, 561), (16, 3, 1, 1327, 12, 80, 0, 0, 0, 1947, 1334),
    (16, 3, 0, 2151, 10, 70, 0, 0, 0, 2772, 1584), (16, 2, 1, 191, 7, 90, 0, 0, 0, 143, 95), (16, 2, 0, 39, 10, 80, 0, 0, 0, 70, 32),
    (16, 3, 1, 84.31, 2, 0, 0, 1, 0, 171.4, 87), (16, 3, 1, 139.4, 2, 0, 0, 1, 0, 237, 120.3),
    (32, 2, 1, 904.98, 1, 0, 0, 1, 0, 688, 442), (16, 3, 1, 94.7, 5, 40, 0, 1, 0, 339, 184.9),
]


def test_the_cheaper_way_of_measured_runs_is_taken(tmp_path):
    """Passes with one mean per group or rounds one by one, priced with the LDS that the launch takes."""
    got = plans(tmp_path, [row[:9] for row in WAYS])
    wrong = [(row, g) for row, g in zip(WAYS, got, strict=True) if g[2] != (row[10] < row[9]) or not g[3]]
    assert not wrong, wrong


INSTANCE = r"""
#include <cstdio>
#include "pass_rules.h"
using namespace moshpit;
int main()
{
    int M, d, dtype, rounds, down, skip, curve, refresh;
    long long P, stride, offset;
    double p;
    while (std::scanf("%d %d %d %lld %lld %lld %d %lf %d %d %d %d", &M, &d, &dtype, &P, &stride, &offset, &rounds, &p, &down, &skip, &curve, &refresh) == 12) {
        int64_t N = 1;
        for (int q = 0; q < d; ++q) N *= M;
        GridAsk a;
        a.absent = p > 0.0;
        a.distortions = curve != 0;
        a.refresh = refresh != 0;
        a.rounds = rounds;
        const Participation who = a.absent ? independent_presence((1.0 - p) / (1.0 + p * (down - 1)), M, skip != 0) : Participation{};
        a.averaged = who.averaged;
        a.live = who.groups;
        GridPlan g;
        const void *at = reinterpret_cast<void *>(4096 + offset * (dtype == 0 ? 4 : 2));
        if (!plan_grid(dtype, N, M, d, P, stride, at, 0, a, &g) || !g.means) {
            std::printf("none\n");
            continue;
        }
        const MeanKernel k = mean_kernel(g, a.absent, a.distortions);
        std::printf("%s %d x %d|%d %d %d %d %d %d\n", k.tab == kClosed ? "closed" : k.tab == kLds ? "lds" : k.tab == kAheadOnly ? "ahead" : "bits", g.phases,
                    g.part, dtype, k.split, k.half, k.nt, k.dist, k.tab);
    }
}
"""

BUILT = r"""
#include <cstdio>
#include <initializer_list>
#include "grid_plan.h"
using namespace moshpit;
int main()
{
    for (int dtype : {0, 1})
        for (int split : {1, 2, 4})
            for (int half : {0, 1, 2, 32})
                for (int nt : {0, 1})
                    for (int dist : {0, 1})
                        for (int tab : {kClosed, kLds, kAheadOnly, kBits})
                            if (mean_kernel_built(dtype, split, half, nt != 0, dist != 0, tab))
                                std::printf("%d %d %d %d %d %d\n", dtype, split, half, nt, dist, tab);
}
"""


def test_the_gpu_tests_take_every_kernel(tmp_path):
    """The runs that test_gpu_mean_rounds.py compares with single rounds go where they say, and together through every instance."""
    import test_gpu_mean_rounds as gpu
    runs = [(M, d, dtype, P, *gpu.layout(M ** d, P, dtype, where), rounds, p, 2, skip, curve, refresh, kernel)
            for M, d, P, dtype, where, p, rounds, refresh, skip, curve, kernel in gpu.FAILURES]
    runs += [(M, d, dtype, P, *gpu.layout(M ** d, P, dtype, where), rounds, 0.0, 1, 0, curve, 0, "closed " + parts if parts and not dtype else None)
             for M, d, P, where, rounds, parts in gpu.EVERYBODY for dtype in (0, 1) for curve in (0, 1)]
    runs += [(M, d, dtype, P, *gpu.layout(M ** d, P, dtype, where), rounds, p, 1, 0, 1, refresh, None)
             for M, d, P, dtype, where, p, rounds, refresh in gpu.LONG_CURVES]
    text = "".join(" ".join(str(int(v) if isinstance(v, bool) else v) for v in run[:-1]) + "\n" for run in runs)
    out = run_host(tmp_path, INSTANCE, text).stdout.splitlines()
    assert len(out) == len(runs)
    wrong = [(run, got) for run, got in zip(runs, out) if got == "none" or (run[-1] is not None and got.split("|")[0] != run[-1])]
    assert not wrong, "\n".join(map(str, wrong))
    built = set(run_host(tmp_path, BUILT).stdout.splitlines())
    taken = {got.split("|")[1] for got in out}
    assert taken == built, sorted(built - taken)


RUNS = r"""
#include <cstdio>
#include <vector>
#include "grid_plan.h"
using namespace moshpit;

int main()
{
    for (int32_t about : {32, 64, 256})
        for (int64_t tiles = 1; tiles < 400 * about; tiles += tiles < 3000 ? 1 : 37) {
            const int32_t run = die_run_of(tiles, about);
            const int64_t span = 8 * int64_t(run), rest = tiles % span;
            const bool few = tiles < 6 * about, many = tiles >= 256 * about;
            if (run < 1 || run > about * 5 / 4) return std::printf("run %d of %lld tiles\n", run, (long long)tiles), 1;
            // (the best of about / 2 + 1 lengths leaves no more than the one asked for)
            if (few ? (tiles >= 16 && rest >= 8) : many ? run != about : rest > tiles % (8 * int64_t(about)))
                return std::printf("run %d of %lld tiles leaves %lld\n", run, (long long)tiles, (long long)rest), 1;
            // the order in which a kernel takes tiles (tile_of) has every tile once
            std::vector<char> seen(tiles, 0);
            for (int64_t i = 0; i < tiles; ++i) {
                const int64_t q = i / span, r = i - q * span, at = run == 1 || (q + 1) * span > tiles ? i : q * span + (r & 7) * run + (r >> 3);
                if (at < 0 || at >= tiles || seen[at]++) return std::printf("tile %lld of %lld\n", (long long)at, (long long)tiles), 1;
            }
        }
    return 0;
}
"""


def test_runs_of_tiles_per_die(tmp_path):
    got = run_host(tmp_path, RUNS)
    assert got.returncode == 0, got.stdout


QUOTIENTS = r"""
#include <cstdio>
#include <cstring>
#include "grid_plan.h"
using namespace moshpit;

int main()
{
    long bad = 0, plain = 0;
    uint64_t x = 0x1234567;
    const auto draw = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x; };
    for (int64_t n = 1; n <= kGridMaxPeers; ++n) {
        const double inv = 1.0 / static_cast<double>(n);
        const auto check = [&](double a) {
            const double want = a / static_cast<double>(n), got = over(a, static_cast<double>(n), inv);
            if (std::memcmp(&want, &got, 8) != 0 && ++bad < 20) std::printf("%a / %lld: %a, not %a\n", a, (long long)n, got, want);
            plain += a * inv != want;
        };
        // squares of sums of differences of binary32 numbers, and the neighbours of products with n (quotients near a tie)
        for (int k = 0; k < 3000; ++k) {
            const uint64_t bits = ((1023 - 300 + draw() % 560) << 52) | (draw() >> 12);
            double a;
            std::memcpy(&a, &bits, 8);
            check(a);
            check(a * a);
            check(nextafter(a * static_cast<double>(n), 0.0));
            check(nextafter(a * static_cast<double>(n), HUGE_VAL));
        }
        check(0.0);
    }
    std::printf("%ld wrong; %ld products with the reciprocal are\n", bad, plain);
    return bad != 0 || plain == 0;
}
"""


def test_distortions_divide_by_the_peers(tmp_path):
    """What a pass subtracts from the squares is the rounded quotient by N, as everywhere else, not a product with 1 / N."""
    out = run_host(tmp_path, QUOTIENTS)
    assert out.returncode == 0, out.stdout
