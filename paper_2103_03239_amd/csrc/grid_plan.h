// Plans of whole-grid passes (grid_rounds.hip, mean_rounds.hip): does a state's shape qualify, how is it
// cut into tiles, which of the two kernels takes them and what lies where in its LDS.  Host arithmetic on
// plain numbers, without GPU types.
#pragma once

#include <math.h>
#include <stdint.h>

namespace moshpit {

constexpr int kPhaseSlots = 8;               // 16-byte slots of the tile in LDS per thread
constexpr int kLdsPerBlock = 80 * 1024;      // two blocks share a compute unit
constexpr int64_t kGridMaxPeers = 4096;
constexpr int kRcpBytes = 272;       // 65 reciprocals, padded to a multiple of 16 bytes
constexpr int32_t kLeastLdsPart = 64;        // bytes of a row in LDS from which on a round's tables take one register or less

// Several rounds on a whole grid of up to 4096 peers in one pass over HBM (grid_rounds.hip).
// plan_grid: does the shape qualify, and how is it cut into tiles (a pure function of its
// arguments; depends on t0 through the first axis only).  The caller fills in the rest.
constexpr int kGridMaxAxes = 12;
struct GridPlan {
    int32_t N, M, d, groups;
    int32_t Wb, wv_shift;            // bytes of a row per tile; log2 of its 16-byte vectors
    int32_t threads, tile_bytes, lds_bytes, red_offset;
    int32_t pad;                     // LDS bytes added after every M rows (bank conflicts of axis 0)
    int32_t die_run;                 // consecutive tiles per die (1: tiles dealt in order)
    int32_t streaming;               // 1 = non-temporal loads and stores
    int32_t phases, max_rounds;      // column parts of a tile (1 or 2); most rounds of one pass
    int32_t axis0;                   // axis of the pass's first round
    uint32_t full_bitmap, magic_m;
    int32_t S[kGridMaxAxes], pad_step[kGridMaxAxes];
    uint32_t magic_s[kGridMaxAxes];
    int64_t row_bytes, valid_bytes, tiles;
    double peers, inv_n;             // N, 1 / N
    // means != 0: the kernel of mean_rounds.hip, and where its LDS holds what
    int32_t means;
    int32_t split;                   // lanes that share a group
    int32_t bits;                    // 1 = who takes part comes as bits instead of places
    int32_t part;                    // bytes of a row in LDS
    int32_t means_at, means_bytes, zero_at, rcp_at, words_at;
    int32_t words_shift;             // log2 of N / 2: 32-bit words that a round's places take
    int32_t sharers;                 // waves that share a distortion (with tables in LDS half of them, an even number)
    int32_t dist_barrier;            // a barrier behind every distortion (a refresh, or LDS has room for one round's terms only)
    int32_t mean_step[kGridMaxAxes];      // bytes between the means that the rows of a group were given by the round before
    // filled in by the caller
    int32_t rounds;
    int32_t dist_before, refresh_first;   // distortion before the first round; refresh before it
    float gamma;
    float step_zero;                 // added to the result of a binary32 step: +0 or -0
    const uint32_t *bitmaps;         // [rounds][groups], device; nullptr = everybody takes part
    const uint8_t *flags;            // [N], device: bit 0 written back, bit 1 takes the local step; nullptr = 3
    const uint32_t *copies;          // [rounds][N] pairs donor << 16 | returning peer; nullptr = no refresh
    const int32_t *copy_counts;      // [rounds]
    const char *grad;                // gradients (SGD) or nullptr
    int64_t grad_row_bytes;
    double *partials;                // [rounds + 1][tiles * phases], of this pass, or nullptr (no distortion wanted)
    uint64_t dist_after;             // bit r: the distortion after round r of the pass is wanted
    // means != 0, with failures: this pass's part of the tables below
    const uint32_t *entries, *moves, *move_rows, *move_bytes, *terms;
    const int32_t *move_counts, *term_counts;
    const uint16_t *places;
};
// What a run asks of its passes.
struct GridAsk {
    bool absent = false;             // somebody may be (a failure schedule)
    bool local_step = false;         // it starts with one
    bool refresh = false;            // returning peers copy another one
    bool distortions = false;        // they are wanted
    int32_t rounds = 0;
    double averaged = 1.0, live = 1.0;       // of the peers, those averaged in a round; of the groups, those with an average
};

// ---- LDS of the kernel that keeps one mean per group ---------------------------------------------

inline int64_t mean_place_stride(const GridPlan &p) { return static_cast<int64_t>(p.threads) * kPhaseSlots * p.phases; }

// a / n, rounded once, for a whole n and inv = 1 / n: two multiply-adds after the product instead of a division (Markstein,
// "Computation of elementary functions on the IBM RISC System/6000 processor", 1990: a quotient within an ulp and a rounded
// reciprocal give the rounded quotient).
#ifdef __HIPCC__
__host__ __device__
#endif
inline double over(double a, double n, double inv)
{
    const double q = a * inv;
    return fma(fma(-q, n, a), inv, q);
}

// The distortions' LDS: the sums of the waves that share one (a half of the block's, the halves in turn; one of each where there is one
// wave), a column each and one of squares, and the totals of a pass.
inline int64_t dist_sums_bytes(int64_t waves, int64_t sharers, int64_t columns, int64_t rounds)
{
    return (waves > 1 ? 2 : 1) * sharers * (columns + 1) * 8 + (rounds + 1) * 8;
}

// How many share it.  Of an odd number of waves one takes none (when all of them did, with two rounds' sums: 12 x 12 bfloat16 of 1 GB, 5
// waves, had 2 blocks a compute unit, 30 rounds 4,830 us, and has 3, 3,150; 13 x 13 x 13 binary32 took two column parts instead of
// one, 10 rounds 2,010 -> 1,130; 20 x 20 of 1 GB, 30 rounds 2,840 -> 2,200).  One less where that makes room for passes of 24 rounds (13 x 13 x 13
// binary32, 3 of 9 waves, 24 rounds of 1 GB in one pass 2,010 us, in two with 4 waves 2,640; 16 x 16 bfloat16, 3 of 8 waves, which leave one
// column part room, where 4 took two: 10 rounds of 1 GB 1,148 -> 1,005, of 100 MB 145 -> 143).
inline int32_t dist_sharers(int64_t waves, int64_t columns, int64_t room)
{
    const int32_t half = waves > 1 ? static_cast<int32_t>(waves / 2) : 1;
    return half > 1 && dist_sums_bytes(waves, half, columns, 24) > room && dist_sums_bytes(waves, half - 1, columns, 24) <= room ? half - 1 : half;
}

// two rounds' places and moves, and the terms of one or two distortions
inline int64_t mean_words_bytes(const GridPlan &p, bool tables, bool distortions)
{
    if (p.bits) return 8 * p.groups;                         // (two rounds' bits)
    return tables && p.part >= kLeastLdsPart ? (!distortions ? 12ll : p.dist_barrier ? 16ll : 20ll) << p.words_shift : 0;
}

// The LDS of a tile of p.N rows x `part` bytes with its two arrays of means; p.part, p.pad, p.split and the
// places in LDS are set.  tables: somebody may be absent; distortions: they are wanted.  Returns the bytes before the distortion's sums.
inline int64_t lay_out_means(GridPlan *p, int32_t part, bool tables, bool distortions)
{
    p->part = part;
    p->split = p->M <= 8 ? 1 : p->M <= 16 ? 2 : 4;
    p->pad = part < 256 && p->M >= 8 && (p->M * part) % 256 == 0 ? part : 0;
    const auto padded_bytes = [&](int64_t rows) { return rows * part + (rows + p->M - 1) / p->M * p->pad; };
    p->tile_bytes = static_cast<int32_t>(padded_bytes(p->N));
    p->means_at = p->tile_bytes;
    p->means_bytes = static_cast<int32_t>(padded_bytes(p->groups));
    p->zero_at = p->means_at + 2 * p->means_bytes;
    const int64_t pad = p->pad;
    int64_t S = 1;
    for (int32_t a = 0; a < p->d; ++a) {
        // groups of the round before that hold the rows of a group of this axis: step from row to row
        const int64_t groups_step = a > 0 ? S / p->M : p->d > 1 ? 1 : 0;
        p->mean_step[a] = static_cast<int32_t>(groups_step * part + groups_step / p->M * pad);
        S *= p->M;
    }
    p->rcp_at = p->zero_at + part;
    // (reciprocals of 0 .. M and no more: with 36 of them 256 peers in tiles of 128 bytes fitted a compute unit three times
    // instead of four: 16 x 16 of 33 MB with failures, 5 rounds 23.5 against 20.7 us, bfloat16 26.1 : 24.3, 100 MB, 16 rounds 77.2 : 68.3)
    p->words_at = p->rcp_at + (tables ? 4 * (8 * p->split + 4) : 0);
    p->words_shift = 0;
    while (2 << p->words_shift < p->N) ++p->words_shift;
    return p->words_at + mean_words_bytes(*p, tables, distortions);
}

// LDS of a pass of `rounds` rounds; tables: p.entries will be set; sums_at: where the distortion's begin.
inline int64_t means_lds_bytes(const GridPlan &p, bool tables, int32_t rounds, bool dist, int64_t esize, int32_t *sums_at)
{
    int64_t at = p.words_at + mean_words_bytes(p, tables, dist);
    *sums_at = static_cast<int32_t>(at);
    const int64_t waves = p.threads / 64;
    if (dist) at += dist_sums_bytes(waves, p.sharers, p.part / esize, rounds);
    return at;
}

// Its tables for `rounds` rounds in passes of pass_rounds, in 32-bit words from the start of a buffer: [entries][with bits: rows that
// move][final places of each pass][moves][terms, where distortions are wanted][move counts][term counts][bitmaps under
// group-skip].  Pieces that are read 16 bytes at a time come first.
struct MeanTableWords {
    int64_t entries, move_rows, move_bytes, places, moves, terms, move_counts, term_counts, bitmaps, total;
};
inline MeanTableWords mean_table_words(const GridPlan &p, int64_t rounds, int64_t pass_rounds, bool terms, bool group_skip)
{
    MeanTableWords w{};
    int64_t at = 0;
    const auto take = [&](int64_t words) { const int64_t mine = at; at += words; return mine; };
    w.entries = take(p.bits ? rounds * p.groups : rounds * p.groups * p.split * 4);
    w.move_rows = take(p.bits ? (rounds + 15) / 16 * 8 * p.threads : 0);
    w.move_bytes = take(p.bits ? (rounds + 15) / 16 * 4 * p.threads : 0);
    w.places = take((rounds + pass_rounds - 1) / pass_rounds * mean_place_stride(p) / 2);
    w.moves = take(rounds * p.N);
    w.terms = take(terms ? rounds * (p.N + p.groups) : 0);
    w.move_counts = take(rounds);
    w.term_counts = take(rounds);
    w.bitmaps = take(group_skip ? rounds * p.groups : 0);
    w.total = at;
    return w;
}

// Which instance of the kernel takes a pass.  half: lanes between the two column parts of a tile, 0 = one part; tab: where the
// places come from (mean_rounds.hip).
constexpr int kClosed = 0, kLds = 1, kAheadOnly = 2, kBits = 3;
struct MeanKernel {
    int split, half, tab;
    bool nt, dist;
};
inline MeanKernel mean_kernel(const GridPlan &p, bool tables, bool dist)
{
    const bool wide = p.part >= kLeastLdsPart;
    MeanKernel k;
    k.split = p.split;
    k.half = p.phases == 1 ? 0 : wide ? 32 : p.part == 32 ? 2 : 1;
    k.tab = !tables ? kClosed : p.bits ? kBits : wide ? kLds : kAheadOnly;
    k.nt = p.streaming != 0;
    k.dist = dist;
    return k;
}
// Those that some plan asks for: rows of less than a cache line are never streamed; grids with tables have 8^d, 16^d or 32^d
// peers, of which 256 fit one part, and 4096 two parts of 16 bytes or one; groups of more than 16 mean at most 1024 peers; distortions of
// wide bfloat16 rows under failures go to the kernel with M copies of a mean.
constexpr bool mean_kernel_built(int dtype, int split, int half, bool nt, bool dist, int tab)
{
    if (tab == kBits) return split == 2 && half <= 1 && !nt && !dist;
    if (tab == kAheadOnly) return !nt && (half == 0 || (split == 2 && half == 1));
    if (tab == kLds) return !(dtype == 1 && dist) && (half == 0 ? split == 2 || !nt : half == 32 && split != 2);
    return half == 0 || half == 32 || (split != 4 && !nt);
}

// ---- LDS of the kernel with M copies of a mean ---------------------------------------------------

inline int64_t bitmap_bytes(int32_t M) { return M <= 16 ? 2 : 4; }

// Sums of a distortion: rows of 256 bytes and more in one part are taken 4 bytes a thread, in `parts` parts of the rows that add
// their columns up in LDS; of others every wave has all columns.  (A tile of few rows and 1 KiB of each left 3 blocks of 5 on a
// compute unit room next to sums by waves.)
#ifdef __HIPCC__
__host__ __device__
#endif
inline int32_t dist_parts(int32_t threads, int32_t row_bytes) { return threads >= row_bytes / 4 ? threads / (row_bytes / 4) : 1; }
#ifdef __HIPCC__
__host__ __device__
#endif
inline int32_t dist_sum_rows(int32_t threads, int32_t row_bytes, int32_t phases)
{
    if (phases > 1 || row_bytes < 256) return threads / 64;
    const int32_t parts = dist_parts(threads, row_bytes);
    return parts > 1 ? parts : 0;
}
inline int64_t copies_sums_bytes(const GridPlan &p, int64_t esize)
{
    const int32_t part = p.Wb / p.phases;
    return (dist_sum_rows(p.threads, part, p.phases) * (part / esize) + p.threads / 64) * 8;
}

inline int64_t copies_lds_bytes(const GridPlan &p, int32_t rounds, bool dist, int64_t esize, int32_t *sums_at)
{
    int64_t at = p.tile_bytes + static_cast<int64_t>(rounds) * p.groups * bitmap_bytes(p.M) + p.N;
    at = (at + 15) / 16 * 16;
    *sums_at = static_cast<int32_t>(at);
    if (dist) at = (at + copies_sums_bytes(p, esize) + 15) / 16 * 16;
    return at + kRcpBytes + 32;
}

// Blocks with so much LDS that share a compute unit: 160 KiB are handed out in 128 pieces.
inline int64_t blocks_by_lds(int64_t bytes) { return 128 / ((bytes + 1279) / 1280); }

// ---- which kernel, which tiles ---------------------------------------------------------------------

// One mean per group (mean_rounds.hip) or M copies of it (grid_rounds.hip)?  MI355X, the former
// against the latter, us:
//   nobody ever absent: ahead from 4 rounds on (16 x 16, 200 MB binary32, 6 rounds 70 : 80; 24 x 24, 1.5 GB bfloat16
//     887 : 1,234; 32 x 32, 16 GB, 16 rounds 10,450 : 14,200), behind by up to 11 % for 2 or 3 (8 x 8 x 8, 1.5 GB
//     bfloat16 715 : 643), by 3 to 9 % for 4 of 32 x 32 in binary32 (250 MB 108 : 99) and for small states of 8 x 8 peers in bfloat16 (8 MB, 8 rounds 12.8 : 12.5);
//     with distortions ahead from the first round in one part (8 x 8 x 8, 1 GB binary32, 5 rounds 660 : 838; two parts: see copies_ahead).  Groups of 2 to 4 save little.
//   with failures, whose tables cost a launch and a wait: ahead from 5 rounds (4 on more than 1024 peers) of
//     states beyond 32 MB on (32 x 32, 16 GB, 8 rounds 8,110 : 9,320, 4 rounds of 200 MB 85 : 83; 16 x 16 x 16, 1.5 GB
//     bfloat16, 4 rounds 911 : 1,222, 16 rounds 1,570 : 2,640; 8 MB, 8 rounds 31 : 28; not taken although ahead: longer runs
//     of small states, 8 MB, 16 rounds 38 : 54), and not for 8 x 8 peers, whose passes
//     wait for memory (1.5 GB binary32, 8 rounds 652 : 631).  Places are 8 to a lane: groups of 8, 16 or 32.  The
//     distortion of bfloat16 rows of 64 bytes and more spills and is not built next to tables (time of M copies over it, 33 to 240 MB, 5 to 40
//     rounds: 256 peers with 5 % absent 1.27 to 1.55, 20 % 1.07 to 1.35, 50 % 0.99; 1,024 with 20 % 1.5 to 1.7, 80 % 0.98; 512 of 0.5 to 2 GB 20 % 0.76 to 0.90).
// A local step would take its registers: not with one.  Where both have a plan copies_ahead looks closer.
inline bool choose_means(GridPlan *p, int64_t esize, const GridAsk &ask)
{
    const int64_t state = p->N * p->row_bytes;
    const bool large = state >= 32000000;
    if (p->M <= 4 || ask.local_step) return false;
    if (ask.absent) {
        if (!large || p->N < 256 || ask.rounds < (p->N > 1024 ? 4 : 5)) return false;
    } else if (!ask.distortions) {
        if (ask.rounds < (esize == 4 && p->N >= 1024 && p->M > 16 && state > 100000000 ? 5 : 4)) return false;
        if (p->M <= 8 && p->N <= 64 && esize == 2 && !large) return false;
    }
    const bool cached = static_cast<double>(p->N) * p->row_bytes <= 256.0 * (1 << 20);
    for (int32_t wb = p->Wb, phases = p->phases; phases <= 2 && wb / phases >= 16;) {
        GridPlan q = *p;
        const int32_t part = wb / phases;
        q.Wb = wb;
        q.phases = phases;
        const int64_t threads = (q.N * part / (16 * kPhaseSlots) + 63) / 64 * 64, waves = threads / 64 < 1 ? 1 : threads / 64;
        q.bits = ask.absent && !ask.refresh && !ask.distortions && part == 16 && q.M == 16 && 2 * q.groups == threads ? 1 : 0;
        const auto fits = [&](bool barrier) {
            q.dist_barrier = barrier ? 1 : 0;
            const int64_t bytes = lay_out_means(&q, part, ask.absent, ask.distortions);
            q.red_offset = static_cast<int32_t>(bytes);
            q.sharers = ask.absent && part >= kLeastLdsPart ? static_cast<int32_t>(waves / 2) : dist_sharers(waves, part / esize, kLdsPerBlock - bytes);
            return bytes + (ask.distortions ? dist_sums_bytes(waves, q.sharers, part / esize, 4) : 0) <= kLdsPerBlock;
        };
        const bool room = (!(ask.distortions && ask.refresh) && fits(false)) || fits(ask.distortions);
        if (ask.absent && (q.M != 8 * q.split || (phases == 2 && part == 32) || (ask.distortions && esize == 2 && part >= 64))) return false;
        // (bfloat16 curves with nobody absent over groups of up to 8, beyond the last-level cache: in two parts 16 waves share a compute unit,
        // in one 14 or 12.  us, one part : two: 6 x 6 x 6 of 300 MB, 2 rounds 198 : 196, of 1 GB, 10 rounds 1,450 : 1,372; 7 x 7 x 7 of 300 MB,
        // 5 rounds 326 : 310, of 1 GB, 2 rounds 636 : 587, 30 rounds 4,050 : 3,540, but 1 round 544 : 683; of 150 MB, 5 rounds 183 : 184)
        const bool halve = ask.distortions && !ask.absent && esize == 2 && q.M <= 8 && !cached && phases == 1 && ask.rounds >= 2 &&
                           blocks_by_lds(q.red_offset + dist_sums_bytes(waves, q.sharers, part / esize, 4)) <= 2;
        if (room && !halve) {
            q.means = 1;
            *p = q;
            return true;
        }
        // (a state in the last-level cache: narrower tiles, see below; 8 x 8 x 8 peers, 8 MiB, 3 rounds: two parts 13.2 us)
        if (cached && phases == 1 && wb > 32) wb >>= 1;
        else ++phases;
    }
    return false;
}

// Consecutive tiles per die, about as many as asked for.  Tiles that whole runs of all dies leave at the end are dealt in order, which costs
// most where tiles share cache lines: of 4096 rows of 100 MB 250 of 762 tiles, 6 rounds 99 us, in runs of 31 (18 left) 74; 1024 rows of
// 60 MB 33.9 -> 30.1.  From 256 runs a die on they are less than 3 % of the tiles, and 32 is the better run (4096 rows of 4.3 GB
// with refresh, 128 of 32,640 tiles left, 2.81 ms; in runs of 34, none left, 3.05).
inline int32_t die_run_of(int64_t tiles, int32_t about)
{
    if (tiles < 6 * about) return tiles >= 16 ? static_cast<int32_t>(tiles / 8) : 1;
    int32_t best = about;
    if (tiles < 256 * about)
        for (int32_t run = about * 3 / 4; run <= about * 5 / 4; ++run)
            if (tiles % (8 * run) < tiles % (8 * best)) best = run;
    return best;
}

// The rest of a plan whose tiles and kernel are chosen.
inline bool fill_in(GridPlan *plan, const void *X, int64_t esize, const GridAsk &ask)
{
    GridPlan &p = *plan;
    const int32_t wb = p.Wb, M = p.M;
    const int64_t N = p.N;
    p.wv_shift = 0;
    while ((16 << p.wv_shift) < wb) ++p.wv_shift;
    const int32_t part = wb / p.phases;              // bytes of a row in LDS
    p.threads = static_cast<int32_t>((N * part / (16 * kPhaseSlots) + 63) / 64 * 64);
    if (p.threads < 64) p.threads = 64;
    if (p.threads > (p.phases == 1 ? 1024 : 512)) return false;
    if (!p.means) {
        p.pad = part < 256 && M >= 8 && (M * part) % 256 == 0 ? part : 0;
        p.tile_bytes = static_cast<int32_t>(N * part + p.groups * p.pad);
    }
    const auto magic = [](int64_t n) { return static_cast<uint32_t>(((int64_t(1) << 32) + n - 1) / n); };
    p.magic_m = magic(M);
    int32_t S = 1;
    for (int32_t a = 0; a < p.d; ++a) {
        p.S[a] = S;
        p.magic_s[a] = S > 1 ? magic(S) : 0;
        p.pad_step[a] = a == 0 ? 0 : S / M * p.pad;
        S *= M;
    }
    p.tiles = (p.valid_bytes + wb - 1) / wb;
    // Tiles of whole cache lines are not seen again: non-temporal (256 rows of 4 MiB: 5.5 TB/s
    // against 5.1 with ordinary accesses).  Others share lines with their neighbours in the row.
    // Runs per die: where tiles share lines, and for rows of one line (1024 rows of 16 MiB, 8
    // rounds: 9.43 -> 9.33 ms, 4 rounds: 10.2 -> 8.3 ms); wider ones lose 1 % to them.
    const bool whole_lines = wb >= 128 && reinterpret_cast<uintptr_t>(X) % 128 == 0 && p.row_bytes % 128 == 0;
    const double state_bytes = static_cast<double>(N) * p.row_bytes;
    const bool cached = state_bytes <= 256.0 * (1 << 20);
    // States in the last-level cache stay there with ordinary accesses (16 x 16 peers, 4 rounds:
    // 128 MiB 58.6 -> 52.8 us, 250 MiB 113 -> 89); below the L2s' 32 MiB the non-temporal ones are
    // ahead again (16 MiB: 12.5 against 13.8), they leave no dirty lines to be written back at the end.
    p.streaming = whole_lines && (!cached || state_bytes <= 24.0 * (1 << 20)) ? 1 : 0;
    // Rows a multiple of 256 KiB apart meet in the same memory channels, and dies that are further apart in the row spread over more of
    // them: 4096 rows, 6 rounds, runs of 32 : 256, 1.1 GB binary32 676 : 640 us, 2.1 GB bfloat16 1,298 : 1,201, with refresh 1,613 :
    // 1,462; 1024 rows in runs of 32 : 64, 0.5 GB 270 : 258, 16 GB 8,700 : 8,470 (256 8,780).  Others: 4096 rows of 262,208
    // 32 : 256 1,180 : 1,187, of 49,152 binary32 567 : 606.
    const bool same_channels = p.row_bytes % (256 * 1024) == 0;
    p.die_run = whole_lines && wb > 128 ? 1 : die_run_of(p.tiles, same_channels && wb <= 32 ? 256 : same_channels && wb <= 128 ? 64 : 32);
    // rounds of one pass: as many bitmaps as fit next to the tile
    const int64_t waves = p.threads / 64, columns = part / esize;
    if (p.means) {
        const int64_t most = ask.distortions ? (kLdsPerBlock - p.red_offset - dist_sums_bytes(waves, p.sharers, columns, -1)) / 8 - 1 : 64;
        p.max_rounds = static_cast<int32_t>(most < 64 ? most : 64);
        return p.max_rounds >= 4;
    }
    const int64_t room = kLdsPerBlock - p.tile_bytes - N - copies_sums_bytes(p, esize) - kRcpBytes - 64;
    const int64_t most = room / (static_cast<int64_t>(p.groups) * bitmap_bytes(M));
    p.max_rounds = static_cast<int32_t>(most < 64 ? most : 64);
    if (p.max_rounds < 4) return false;      // (2^12 peers; 24 x 24 in tiles of 128 bytes with 8 columns to a vector)
    return true;
}

// Of two plans for a state, is the one with M copies of a mean the faster?  MI355X, one mean against M copies, us, binary32
// unless stated.
inline bool copies_ahead(const GridPlan &copies, const GridPlan &means, int64_t esize, const GridAsk &ask)
{
    const int32_t M = copies.M, rounds = ask.rounds;
    const bool f32 = esize == 4;
    // Bitmaps of all groups next to the tile leave M copies fewer rounds to a pass (16 x 16 x 16 peers 14, 8 x 8 x 8 24 to 40): a pass more
    // is never worth it (16 x 16 x 16 of 0.98 GB, group-skip with 5 % absent, 16 rounds 1,240 : 1,920).
    const auto passes = [&](const GridPlan &p) { return (rounds + p.max_rounds - 1) / p.max_rounds; };
    if (passes(copies) > passes(means)) return false;
    // With failures a short run of a small state does not make up for its larger tables, which take the launch that fills
    // them longer (40 MB: 16 x 16 x 16, 5 rounds 50.0 : 47.8, 12 rounds 70.0 : 69.9, bfloat16 53.8 : 52.0; 32 x 32, 5
    // rounds 32.5 : 31.6, 48 MB, 8 rounds 41.8 : 43.9; 16 x 16 25.7 : 26.6).
    const int64_t state = copies.N * copies.row_bytes;
    if (ask.absent && !ask.refresh && !ask.distortions && state < 48000000 &&
        rounds < (copies.N > 1024 ? 10 : f32 && M > 16 ? 8 : 0)) return true;
    // Who is absent costs M copies nothing.  Next to the means an absent peer's value moves to its own row (most often where
    // half are away), a group without an average is read through its table all the same, and a distortion takes a term of every
    // absent peer.  Time with one mean per group over that with M copies, 60 to 1,500 MB:
    const bool short_of_time = rounds >= 8 || state < 100000000;
    const double moves = ask.averaged * (1.0 - ask.averaged);
    if (ask.absent && ask.distortions) {
        // (curves of 5 to 40 rounds.  256 peers, 33 to 130 MB: 30 % absent 0.93 to 1.03, 40 % 1.07, 50 % 1.09 to 1.16, from 190 MB on 60 % 0.93, 70 %
        // 0.97 to 0.99, 80 % 1.02, 90 % 1.10 to 1.12; 512: 30 % 0.93 to 0.95, 40 % 1.05 to 1.08, 90 % 1.3 to 2; 1,024 within 256 MiB: 40 % 0.92
        // to 0.97, 50 % 0.97 to 1.04, 60 % 1.04 to 1.11, beyond: 5 % 0.77, 20 % 1.04 to 1.08, 40 % 1.11 to 1.17, 50 % 1.19 to 1.23, 40 rounds 5 % 0.77, 50 % 1.05; 4,096: 40 % 0.68 to
        // 0.99, 60 % 1.02 to 1.11 up to 12 rounds, 24 rounds 0.85, 70 % 1.05 to 1.18, 40 rounds 0.98, 95 % 1.05 to 1.28, bfloat16 80 % 0.90 to
        // 1.06, 90 % 1.00 to 1.15, 95 % 1.03 to 1.10)
        const bool cached = state <= 268435456;
        const double least = M <= 8 ? 0.6 : M > 16 ? (cached ? 0.45 : rounds < 40 ? 0.81 : 0.5)
                             : copies.N <= 1024 ? (state < 130000000 ? 0.65 : 0.25)
                             : f32 ? (rounds < 24 ? 0.45 : 0.15) : rounds < 24 ? 0.15 : 0.0;
        // (with returning peers, whose rows M copies have to move; curves of 5 to 24 rounds by the peers averaged: 512 peers within 256 MiB 54 % 0.89 to
        // 0.97, 43 % 1.00 to 1.07, 33 % 1.07 to 1.22, beyond 54 % 1.22 to 1.28; 256 peers, 38 to 120 MB 67 % 0.93, 54 % 1.02, 43 % 1.06, from 190 MB
        // on 25 % 0.89 to 0.91, 11 % 0.95 to 1.00, 5 % 1.08; 1,024 within 256 MiB 33 % 0.95, 25 % 1.02 to 1.06, beyond 54 % 0.88 to 0.99, 43 % 1.00 to
        // 1.04, 25 % 1.12 to 1.18; 4,096 33 % 0.83 to 0.96, 25 % 1.07, 11 % 1.05 to 1.11, bfloat16 18 % 0.97, 5 % 0.99 to 1.10)
        const double with_refresh = M <= 8 ? (cached ? 0.45 : 0.6) : M > 16 ? (cached ? 0.28 : 0.45)
                                    : copies.N <= 1024 ? (state < 130000000 ? 0.55 : 0.08) : f32 ? 0.28 : 0.1;
        if (ask.averaged < (ask.refresh ? with_refresh : least)) return true;
    } else if (ask.absent && copies.N <= 1024) {
        if (ask.refresh) {
            // (512 peers, 12 rounds: 6 % of the groups live 0.92 to 1.07, 2 % 1.02 to 1.18, 6 rounds of 300 MB and more 0.86 to 0.98)
            if (M <= 8 && ask.live < 0.03 && short_of_time) return true;
        } else {
            // (12 rounds, 512 peers in bfloat16: 50 % of the groups live 0.94 to 0.95, 19 % 1.07 to 1.14, 6 % 1.39, in binary32 50 %
            // 1.00 to 1.04, 43 % of them whole 1.02 to 1.07, 19 % 1.09 to 1.14; 256: 19 % 0.85 to 0.97, none 1.16 to 1.24; 1,024: 46 % 0.83 to
            // 0.90, 3 % 1.06 to 1.10; in binary32, 512 peers, half of them absent 1.04 to 1.12, 30 or 70 % 0.95 to 1.01, 256
            // beyond 256 MiB, 6 rounds 1.04 to 1.07, 12 rounds 0.93 to 0.98)
            if (ask.live < (M > 8 ? 0.1 : f32 ? 0.45 : 0.3) && short_of_time) return true;
            if (f32 && M <= 8 && moves > 0.215) return true;
            if (f32 && M > 8 && M <= 16 && moves > 0.22 && rounds <= 8 && state > 268435456) return true;
        }
    } else if (ask.absent && !ask.refresh && !ask.distortions) {
        // (4,096 peers of 60 MB: 30 % absent 0.98 to 1.00, 50 to 95 % 0.98 to 1.12; with two moves a thread at hand half of the peers
        // are too many for longer runs: bfloat16, 300 MB and more, 6 rounds 0.89, 12 rounds 1.14 to 1.16, at 30 and 70 % 0.98 to 1.01)
        if (ask.averaged < 0.6 && state < 100000000) return true;
        if (means.bits && !f32 && rounds > 8 && moves * copies.N > 1.9 * means.threads) return true;
    }
    // The means cost a second column part that M copies do without.  8 x 8 x 8 peers of 1 GB: 5 rounds 440 : 421, 8 rounds 425 :
    // 502; with failures 5 rounds 457 : 433, 8 rounds 446 : 515 (and refresh: 5 rounds 458 : 554); with failures and curve, where few
    // registers are left, 5 rounds 1,204 : 867, of 3 GB 20 rounds 8,220 : 7,080, 64 rounds 20,270 : 21,460.  Curves with nobody absent: 24 x 24 of 0.3 to 3 GB
    // 1 round 0.81 to 0.83 times as fast, 2 rounds 0.88, 3 rounds 0.96, 5 rounds 1.04 to 1.07, 12 rounds 4,990 : 6,030.
    // (In bfloat16 M copies take longer: 8 x 8 x 8, 5 rounds with failures 460 : 542.)
    if (f32 && copies.phases == 1 && means.phases == 2) {
        if (ask.distortions) {
            if (rounds < (ask.absent ? 40 : M > 16 ? 4 : 0)) return true;
        } else if (M <= 8 && !ask.refresh && rounds < 6) {
            return true;
        }
    }
    // A block with the means takes more LDS.  Where the chip has room for all blocks with M copies at once, but not for all of the
    // others, those come in two turns.  28 MB, nobody absent: 7 x 7 x 7 (2 blocks a compute unit : 3; 640 tiles) 4
    // rounds 22.4 : 19.1, 64 rounds 138 : 127, bfloat16 27.9 : 25.2 (20 MB, one turn of each: 13.7 : 15.8); 8 x 8, 4 rounds 18.6 :
    // 15.9, 10 rounds 24.4 : 22.9, 32 rounds 49.0 : 48.8; 8 x 8 x 8, 4 rounds 18.3 : 15.7, 10 rounds 25.1 : 24.3, 16 rounds 32.0 : 32.7; 24 x 24 of 30 MB, 4 rounds 22.8 : 20.7, 16
    // rounds 45.0 : 43.5; with failures 8 x 8 x 8 of 33 MB, 5 rounds 40.9 : 38.4, 20 rounds 50.3 : 48.8.  Other groups of 9 to 16, other bfloat16 rows and distortions are worth more than a turn (9 x 9 of 33 MB, 4 rounds
    // 20.2 : 24.2; 8 x 8 x 8 bfloat16, 4 rounds 23.2 : 25.2; curve of 8 x 8 x 8, 1 round 43.7 : 40.1, 2 rounds 0.96 times as fast, 5 rounds
    // 53.8 : 56.5).
    const int32_t most = ask.absent ? (f32 && M <= 8 && !ask.refresh && !ask.distortions ? 20 : 0)
                         : ask.distortions ? (f32 && M <= 8 ? 2 : 0) : M == 7 ? 64 : !f32 ? 0 : M > 16 ? 64 : M > 8 ? 0 : copies.N <= 64 ? 10 : 6;
    if (rounds > most) return false;
    int32_t at = 0;
    const auto pass = [&](const GridPlan &p) { return rounds < p.max_rounds ? rounds : p.max_rounds; };
    const int64_t room_copies = 256 * blocks_by_lds(copies_lds_bytes(copies, pass(copies), ask.distortions, esize, &at));
    const int64_t room_means = 256 * blocks_by_lds(means_lds_bytes(means, ask.absent, pass(means), ask.distortions, esize, &at));
    return copies.tiles <= room_copies && means.tiles > room_means;
}

inline bool plan_grid(int dtype, int64_t N, int32_t M, int32_t d, int64_t P, int64_t row_stride, const void *X, int64_t t0,
                      const GridAsk &ask, GridPlan *out)
{
    const int64_t esize = dtype == 0 ? 4 : 2;
    GridPlan p{};
    p.valid_bytes = P * esize;
    p.row_bytes = row_stride * esize;
    if (N > kGridMaxPeers || M > 32 || p.valid_bytes < 16) return false;
    p.N = static_cast<int32_t>(N);
    p.M = M;
    p.d = d;
    p.groups = static_cast<int32_t>(N / M);
    p.peers = static_cast<double>(N);
    p.inv_n = 1.0 / p.peers;
    p.full_bitmap = M == 32 ? ~0u : (1u << M) - 1u;
    p.axis0 = static_cast<int32_t>(t0 % d);
    // Widest tile: rows of 512 bytes beat 1 KiB on 64 rows (2.55 against 2.73 ms), 256 bytes beat
    // 128 on 256 rows (0.40 against 0.46 ms for 3 rounds).
    int32_t wb = 1024;
    while (wb > 256 && N * wb > 32 * 1024) wb >>= 1;
    while (wb > 128 && N * wb > 64 * 1024) wb >>= 1;
    while (wb > 32 && N * wb > 128 * 1024) wb >>= 1;
    // A state of up to 256 MiB stays in the last-level cache and is bound by latency more than by
    // the width of its accesses: 256 bytes at most (250 MiB, 4 x 4 x 4 peers: 103 against 109 us at
    // 512), one part in LDS for up to 1024 peers (32 x 32, 4 rounds: 8 MiB 22 -> 14 us, 250 MiB
    // 115 -> 97) and, above, while that gives a compute unit no second tile to run (16 x 16 x 16,
    // 6 rounds: 16 MiB 46 -> 29 us, but 128 MiB 96 -> 127; rows of whole vectors only, since a
    // last tile of less than 16 bytes takes 16 from its neighbour, which must have more) ...
    const double state_bytes = static_cast<double>(N) * p.row_bytes;
    const bool cached = state_bytes <= 256.0 * (1 << 20);
    if (cached && wb > 256) wb = 256;
    if (cached && N * wb > 64 * 1024 && (N <= 1024 || (p.valid_bytes % 16 == 0 && p.valid_bytes <= 256 * wb))) wb >>= 1;
    // ... and narrow tiles, so that every compute unit gets several blocks (8 MiB, 4 x 4 x 4 peers,
    // 6 rounds: 15.3 -> 13.3 us; 5 x 5 x 5, 32 MiB: 31.9 -> 25.1), but not below 4 KiB or one
    // cache line of 256 rows and more.
    const int32_t least = N >= 256 ? 128 : 64;
    while (wb > least && N * wb > 4096 && (p.valid_bytes + wb - 1) / wb < 2048) wb >>= 1;
    while (wb > 32 && wb / 2 >= p.valid_bytes) wb >>= 1;
    p.Wb = wb;
    p.phases = N * wb > 72 * 1024 ? 2 : 1;
    GridPlan one = p;
    const bool copies = fill_in(&p, X, esize, ask), means = choose_means(&one, esize, ask) && fill_in(&one, X, esize, ask);
    if (!copies && !means) return false;
    *out = means && !(copies && copies_ahead(p, one, esize, ask)) ? one : p;
    return true;
}

}  // namespace moshpit
