// Sizes and choices of multi-round passes: host arithmetic on plain numbers, without GPU types.
#pragma once

#include <math.h>
#include <stdint.h>

#include "grid_plan.h"

namespace moshpit {

// Tables of whole-grid passes (who takes part in which round, who copies whom) are built for a
// bounded number of rounds at a time, so that their memory and the launch that fills them do not
// grow with the length of a run.  16 MiB hold, of 16 x 16 x 16 peers, 16,000 rounds of the kernel with M copies of a mean (with
// refresh 960) and 390 of the kernel that keeps one mean per group, in both cases cut to whole passes.
constexpr int64_t kGridTableBytes = int64_t(16) << 20;
constexpr int64_t kGridTableRounds = 65536;            // (the launch has one block per round)

// Per round: a 32-bit bitmap per group; with refresh a list of at most N pairs and its length.
inline int64_t grid_table_round_bytes(int64_t N, int32_t M, bool refresh)
{
    return 4 * (N / M) + (refresh ? 4 * N + 4 : 0);
}

// Of the kernel that keeps one mean per group, at most (mean_table_words): 16 bytes of places per lane of a group, 4 per peer that
// moves, 4 per term of the distortion, two counts, a bitmap per group.
inline int64_t mean_table_round_bytes(int64_t N, int32_t M, int32_t split)
{
    const int64_t groups = N / M;
    return groups * 16 * split + 4 * N + 4 * (N + groups) + 8 + 4 * groups;
}

// Rounds the tables are built for at once: whole passes of max_rounds rounds, at least one.
inline int64_t table_rounds(int64_t round_bytes, int64_t max_rounds)
{
    int64_t n = kGridTableBytes / round_bytes;
    if (n > kGridTableRounds) n = kGridTableRounds;
    n = n / max_rounds * max_rounds;
    return n < max_rounds ? max_rounds : n;
}
inline int64_t grid_table_rounds(int64_t N, int32_t M, bool refresh, int64_t max_rounds)
{
    return table_rounds(grid_table_round_bytes(N, M, refresh), max_rounds);
}

// A pass leaves one partial sum per tile for every distortion it computes; they are summed before
// the next pass, so the buffer holds those of one pass, and a pass over a state so wide that they
// would take more than 256 MiB takes fewer rounds.
constexpr int64_t kGridPartialBytes = int64_t(256) << 20;

inline int32_t grid_pass_rounds(int32_t max_rounds, int64_t entry_tiles)
{
    if (entry_tiles <= 0) return max_rounds;
    const int64_t n = kGridPartialBytes / (8 * entry_tiles) - 1;
    return n < 1 ? 1 : n < max_rounds ? static_cast<int32_t>(n) : max_rounds;
}

// ---- which way a run goes ---------------------------------------------------------------------
//
// On grids that whole-grid passes serve, a run can take one pass per max_rounds rounds (it reads
// every row of the state and writes those that take part in some round of the pass), or the way
// runs go elsewhere: round by round, a round touching only the rows of groups in which somebody
// is averaged, or (MOSHPIT_RUN_FUSED) sub-grid passes, which touch the rows that take part in them.
// Which is shorter depends on how many peers are away, on the number of rounds, and on the tile:
// MI355X, times of the whole-grid pass against the other way,
//   16 x 16 x 1,048,576 binary32:       2 rounds 408 us against 733 with everybody present, 401 : 597 with
//                                       20 % absent, 260 : 166 with 90 %; 8 rounds, 90 %: 459 : 903
//   32 x 32 x 4,194,304 binary32:       2 rounds, 50 %: 7.4 ms against 6.4; 8 rounds 9.3 : 25.3 ms; 8 rounds of
//                                       group-skip at 20 % (hardly a group is whole): 5.1 : 2.5 ms
//   16 x 16 x 16 x 262,144 bfloat16:    2 rounds, 20 %: 1.65 ms against 1.15; 4 rounds 1.87 : 2.29 ms;
//                                       fused, 2 rounds: 1.65 : 0.86, 8 rounds: 2.2 : 3.2 ms
//   3^7 x 131,072 binary32:             fused, 8 rounds, 20 %: 2.0 ms against 1.17 (tall tiles, narrow rows)
// So both ways are priced and the cheaper one taken.  The figures below were fitted to 3,300 runs
// on 46 grids of 16 to 4096 peers (rows of 0.1 KB to 64 MB, states of 50 KB to 4 GB; 2 to 10
// rounds, 0 to 90 % absent; with and without curve, refresh, group-skip, local step and
// MOSHPIT_RUN_FUSED) so that the choice comes out right: the way taken costs within 5 % of the
// better one in 96 % of them and within 15 % in 98 %; half of the predicted times lie within 12 %
// of the measured ones.  Times are in microseconds, sizes in megabytes (10^6 bytes).

// Who takes part, as fractions: of the peers in a round, of the rows that lie in a group with an
// average (`averaged`) and of the groups that have one.
struct Participation {
    double present = 1.0, averaged = 1.0, groups = 1.0;
    bool failures = false, group_skip = false;
    double ever_seen = -1.0;             // measured fraction of the peers that take part at some time; < 0: unknown
    // of the peers that take part in some one of n rounds
    double ever(double n) const
    {
        if (!failures) return 1.0;
        const double e = 1.0 - pow(1.0 - (group_skip ? averaged : present), n);
        return ever_seen >= 0.0 && ever_seen < e ? ever_seen : e;
    }
};

// Peers present independently with probability q in groups of M.
inline Participation independent_presence(double q, int32_t M, bool group_skip)
{
    Participation w;
    w.failures = true;
    w.group_skip = group_skip;
    w.present = q;
    if (group_skip) {
        w.averaged = w.groups = pow(q, M);
    } else {
        const double others = pow(1.0 - q, M - 1);
        w.averaged = q * (1.0 - others);
        w.groups = 1.0 - (1.0 - q) * others - M * q * others;
    }
    return w;
}

// Masks given by the caller, [rounds][N] bytes: about 128 groups and 64 peers of them are looked at.
inline Participation sampled_presence(const uint8_t *masks, int64_t rounds, int64_t N, int32_t M, int32_t d, int64_t t0,
                                      bool group_skip)
{
    Participation w;
    w.failures = true;
    w.group_skip = group_skip;
    const int64_t groups = N / M, all = groups * rounds, step = all / 128 > 0 ? (all / 128) | 1 : 1;
    int64_t seen = 0, present = 0, averaged = 0, live = 0;
    for (int64_t k = 0; k < all; k += step, ++seen) {
        const int64_t r = k / groups, g = k % groups;
        int64_t S = 1, on = 0;
        for (int64_t q = 0; q < (t0 + r) % d; ++q) S *= M;
        const uint8_t *first = masks + r * N + g / S * S * M + g % S;
        for (int64_t j = 0; j < M; ++j) on += first[j * S] != 0 ? 1 : 0;
        present += on;
        if (on >= 2 && (!group_skip || on == M)) {
            averaged += on;
            ++live;
        }
    }
    w.present = static_cast<double>(present) / static_cast<double>(seen * M);
    w.averaged = static_cast<double>(averaged) / static_cast<double>(seen * M);
    w.groups = static_cast<double>(live) / static_cast<double>(seen);
    const int64_t peer_step = N / 64 > 0 ? N / 64 : 1, round_step = rounds / 64 > 0 ? rounds / 64 : 1;
    int64_t peers = 0, ever = 0;
    for (int64_t i = 0; i < N; i += peer_step, ++peers) {
        bool on = false;
        for (int64_t r = 0; r < rounds && !on; r += round_step) on = masks[r * N + i] != 0;
        ever += on ? 1 : 0;
    }
    // (more rounds than were looked at can only add peers)
    if (round_step == 1) w.ever_seen = static_cast<double>(ever) / static_cast<double>(peers);
    return w;
}

struct RunSize {
    int64_t N = 0, valid_bytes = 0, row_bytes = 0;
    int32_t M = 0, element_bytes = 0;
    double megabytes() const { return 1e-6 * static_cast<double>(N) * static_cast<double>(row_bytes); }
    bool cached() const { return N * row_bytes <= (int64_t(256) << 20); }        // the last-level cache holds the state
};

// One round of the single-round kernel: a launch, a work item per KiB of a group's row (a wave that
// finds nobody to average ends at once; one that does waits for its rows), and the traffic.
inline double single_round_us(const RunSize &z, const Participation &w)
{
    const int32_t vectors = z.M <= 2 ? 4 : z.M > 4 && z.M <= 8 ? 2 : 1;      // KiB of a row per work item
    const double items = 1e-3 * static_cast<double>(z.N / z.M) * static_cast<double>((z.valid_bytes + 1024 * vectors - 1) / (1024 * vectors));
    const double dispatch = z.M <= 2 ? 0.47 : z.M <= 4 ? 0.22 : z.M <= 8 ? 0.63 : z.M <= 16 ? 0.44 : 0.72;
    const double waits = z.M <= 4 ? 0.0 : z.M <= 8 ? 0.12 : z.M <= 16 ? 0.9 : 1.9;
    const double us = items * (dispatch + waits * w.groups) + 2.0 * z.megabytes() * w.averaged * 0.14;
    return 4.0 + us * (z.cached() ? 0.8 : 1.0);
}

// One sub-grid pass over `rounds` rounds.
inline double fused_pass_us(const RunSize &z, const Participation &w, int32_t rounds, bool whole_grid, int32_t blocks_per_cu)
{
    const double bf16 = z.element_bytes == 2 ? 1.7 : 1.0, e = w.ever(rounds);
    const double per_mb = blocks_per_cu == 2 ? 0.053 + 0.21 * e + bf16 * rounds * (0.03 + 0.031 * w.averaged)
                                             : 0.11 + 0.38 * e + bf16 * rounds * 0.024;
    const double cached = z.cached() && whole_grid && blocks_per_cu == 2 ? 0.77 : 1.0;
    return 6.9 + 3.1 * rounds + z.megabytes() * cached * per_mb;
}

// Rounds one by one are taken if they are priced below this part of the passes with M copies of a mean.  Over 22,000 runs on 11
// grids, 256 KiB to 3 GB, they were slower than the passes in 1 of 1,400 runs then (45 % at most); with
// any price below that of the passes in 1 of 40 (up to twice).  It leaves 5 % of the runs more than 5 %
// slower than the better way.
// Passes with one mean per group are taken unless rounds are priced below them: over 801 runs under failures the way taken is
// more than 5 % slower than the better one in 3.0 % and more than 15 % in 1.6 % then, 5.9 and 3.8 % at four fifths.
// So are passes with distortions: over 2,191 curves on 18 grids (0.3 MB to 5 GB, 1 to 40 rounds, 0 to 95 % absent) rounds are taken though a pass is more
// than 5 % faster in 0.9 %, a pass though rounds are in 0.4 % (0.3 and 1.5 % at four fifths; with the prices of the distortions before they
// got cheaper 4.9 and 0.6 %).
constexpr double kRoundsAhead = 0.8, kRoundsAheadOfMeans = 1.0;

// A distortion on its own: two launches and the chain over the rows that a wave walks, or one read of the state where that takes
// longer.  1,024 binary32 rows of 1.6, 25, 100 and 1,600 MB take 7.5, 8.2, 20 and 235 us, 4,096 bfloat16 rows 17, 19, 22 and 236; between
// rounds, whose launches it is queued among, 4 more of a small state.
inline double distortion_us(const RunSize &z)
{
    const double chain = 11.0 + static_cast<double>(z.N) * (z.element_bytes == 2 ? 0.0027 : 0.0015), read = 8.0 + 0.15 * z.megabytes();
    return chain > read ? chain : read;
}

// A refresh on its own: plan, and a copy whose launch is sized for the state.
inline double refresh_us(const RunSize &z) { return 6.5 + 0.14 * z.megabytes(); }

// Whole-grid passes over `rounds` rounds: the tiles' memory traffic by the bytes of a row in a tile
// (narrow ones share cache lines and DRAM pages badly, rows left out of a write most of all), and
// the rounds in LDS: every thread takes `items_per_thread` items a round, one after the other, on
// as many blocks as share a compute unit.  The two hardly overlap.
struct GridTiles {
    int32_t row_bytes = 0, parts = 1, threads = 0, lds_bytes = 0, max_rounds = 1;
    int64_t tiles = 0;
    bool means = false;                  // the kernel that keeps one mean per group; else M copies of it
    bool curve = false;                  // distortions are wanted
};
inline GridTiles grid_tiles(const GridPlan &p, const GridAsk &ask, int64_t esize)
{
    GridTiles t;
    t.row_bytes = p.Wb;
    t.parts = p.phases;
    t.threads = p.threads;
    t.max_rounds = p.max_rounds;
    t.tiles = p.tiles;
    t.means = p.means != 0;
    t.curve = ask.distortions;
    int32_t sums_at = 0;
    t.lds_bytes = p.tile_bytes + p.N;
    if (t.means) t.lds_bytes = static_cast<int32_t>(means_lds_bytes(p, ask.absent, ask.rounds < p.max_rounds ? ask.rounds : p.max_rounds, ask.distortions, esize, &sums_at));
    return t;
}
inline bool rounds_ahead(double by_rounds, double by_passes, const GridTiles &t)
{
    return by_rounds < (t.means || t.curve ? kRoundsAheadOfMeans : kRoundsAhead) * by_passes;
}
inline double grid_passes_us(const RunSize &z, const Participation &w, const GridTiles &t, int32_t rounds, int32_t distortions)
{
    const bool f32 = z.element_bytes == 4;
    const int32_t split = z.M > 16 ? 4 : z.M > 8 && f32 ? 2 : 1;             // lanes that share an item
    const double item_us = z.M > 16 ? 0.73 : z.M > 8 ? (f32 ? 0.69 : 1.2) : z.M > 4 ? (f32 ? 0.76 : 0.87) : z.M > 2 ? 0.48 : 0.22;
    const int64_t items = z.N / z.M * (t.row_bytes / t.parts / (4 * z.element_bytes)) * split;
    const double per_thread = static_cast<double>((items + t.threads - 1) / t.threads);
    const int32_t waves = t.threads / 64;
    int64_t per_cu = waves > 8 && waves <= 12 ? 2 : 16 / waves;              // (75 to 81 registers each in one part)
    if (per_cu > 160 * 1024 / t.lds_bytes) per_cu = 160 * 1024 / t.lds_bytes;
    if (per_cu < 1) per_cu = 1;
    const double turns = static_cast<double>(t.tiles) / (256.0 * static_cast<double>(per_cu));
    // One mean per group, fitted to 1,333 runs (half of the prices lie within 7 % of the times, 90 % within 30): the rounds
    // are a share of what M copies take, and hide half of the memory's time under failures, whose tables take a while to fill.
    const int32_t kind = z.M <= 8 ? 0 : z.M <= 16 ? 1 : 2;
    constexpr double kEverybody[3] = {0.68, 0.62, 0.54}, kLive[3] = {0.19, 0.45, 0.55};
    constexpr double kSome32[3] = {1.19, 1.26, 1.07}, kSome16[3] = {0.74, 0.95, 0.75};
    const bool tables = t.means && w.failures;
    const double share = !t.means ? 0.63 + 0.37 * w.groups : tables ? (f32 ? kSome32 : kSome16)[kind] + kLive[kind] * w.groups : kEverybody[kind];
    const double fixed = tables ? 11.3 + 32.0 * static_cast<double>(z.N) / 4096.0 : 4.2 + 8.2 * static_cast<double>(z.N) / 4096.0;
    const double round_us = (turns > 1.0 ? turns : 1.0) * per_thread * item_us * share * t.parts;
    const bool narrow = t.row_bytes <= 64;
    const double read = t.row_bytes <= 32 ? 0.47 : narrow ? 0.36 : t.row_bytes <= 128 ? 0.25 : 0.17;
    const double masked = t.row_bytes <= 32 ? 0.34 : narrow ? 0.25 : t.row_bytes <= 128 ? 0.12 : 0.13;
    const double whole = t.row_bytes <= 32 ? 0.19 : narrow ? 0.17 : t.row_bytes <= 128 ? 0.13 : 0.11;
    const double memory = z.megabytes() * (z.cached() ? (narrow ? 0.66 : 0.9) : 1.0) * (tables ? 0.49 : 1.0);
    double us = 0.0;
    for (int32_t left = rounds; left > 0; left -= t.max_rounds) {
        const int32_t n = left < t.max_rounds ? left : t.max_rounds;
        us += fixed + memory * (read + (w.failures ? masked * w.ever(n) : whole)) + n * round_us;
    }
    // A distortion, fitted to 2,200 curves: a barrier or two, and the terms of a tile: every row, every group, or groups and absent rows.
    const double away = 1.0 - w.averaged;
    const double latency = !t.means ? (f32 ? 2.0 : 2.3) : tables ? 1.5 : 1.0;
    const double terms = !t.means ? (f32 ? 0.06 : t.row_bytes >= 256 ? 0.107 : 0.135)
                         : tables ? (t.parts == 1 ? 0.006 + 0.115 * away : f32 ? 0.043 + 0.113 * away : 0.051 + 0.149 * away)
                                  : (f32 ? 0.028 : 0.0465) * (t.parts == 1 ? 1.0 : 1.4);
    return us + distortions * (latency + z.megabytes() * terms);
}

}  // namespace moshpit
