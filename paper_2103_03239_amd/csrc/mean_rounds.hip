// Consecutive averaging rounds on a WHOLE grid of up to 4096 peers in one pass over HBM, for
// gfx950, in groups of more than a few peers: the loop of Alg. 1 with the distortion after every round
// (left-hand side of the equation of Thm 3.2), the refresh of returning peers (App. "Training with
// a dynamic number of peers") and the local step of Moshpit SGD (Alg. 2) in between.
//
// Tiles as in grid_rounds.hip (all N rows and Wb bytes of each, in the registers of a block's
// threads, in LDS at most 64 KiB at a time), and the arithmetic of the single-round kernel: balanced
// tree of 16-position blocks, one correctly rounded division, one rounding to the storage type.
//
// What a round costs there is that it reads the tile from LDS and writes it back: M copies of every
// group's mean, each with its own address and its own test of who takes part.  Here a round writes
// ONE mean per group, into one of two arrays of means that take turns, and a peer's value is
// wherever the last round left it: the mean of the group it was averaged in, or, for a peer the
// last round passed over, the row of its own.  Who reads what from where depends on the schedule alone,
// not on the tile, so it is worked out once per run (mean_plan_kernel): per group and round the LDS
// places of its positions (absent ones read zeros) and its count, and the few rows that have to move: a
// peer that was averaged in the last round and is not in this one takes its value back to its own
// row before the array of means it lives in is overwritten.  A returning peer that copies another
// one just reads its row.  A run in which nobody is ever absent has its places in closed form.
//
// A lane takes 8 positions of a group and 16 bytes of a row; SPLIT lanes share a group.  Per 16
// bytes it costs one address (one multiply-add), one 128-bit LDS read and the additions.
//
// The distortion after a round needs one term per group (weight: the count) and one per peer that
// was not averaged, instead of one per peer.  Half of a block's waves take it, the halves in turn, while the others are at the next
// round; lanes are summed by exchanges that halve the columns each keeps, waves by one of them behind the next round's barrier.
//
// What bounds it (MI355X; before: the kernel of grid_rounds.hip).  A round takes 21 us per GiB of
// binary32 where nobody is absent (before 39), 0.42 ms on 32 x 32 peers x 4,194,304 (0.63); on 16 x 16 x 16
// bfloat16 it is the widening and adding, 31 us of 2 GiB (75).  Short runs wait for memory as before:
//   32 x 32 x 4,194,304 binary32, 8 rounds, 20 % absent          9.35 -> 8.11 ms (4.2 TB/s; a copy in tiles of 128
//                                                                bytes 4.7), 16 rounds, nobody 14.2 -> 10.5
//   16 x 16 x 1,048,576 binary32, 10 rounds, 11 distortions      1.54 -> 0.82 ms
//   12 x 12 x 3,472,192 bfloat16, 30 rounds, 31 distortions      4.59 -> 3.15 ms (an odd number of waves, 5)
//   16 x 16 x 16 x 131,072 bfloat16, 6 rounds with refresh       1.12 -> 0.87 ms
//   16 x 16 x 16 x 262,144 bfloat16, 12 rounds, nobody absent    1.98 -> 1.48 ms
//   the same with 10 % absent                                    2.09 -> 1.90
// What a compute unit's time goes into (counters): vector instructions take 89 % of the issue slots on 16 x 16 x 16 bfloat16,
// 61 % under the curve of 16 x 16 binary32 (binary64 sums), 56 % on 32 x 32, where memory moves 4.2 TB/s.
// Next to a second part of the tile few of the 128 registers are free: six of the kernels with the distortion keep 28 to 188
// bytes a lane in scratch, the others none.
// A round's vector instructions count as much as its LDS traffic, and a load from memory in a round costs
// more than either: a compute unit returns loads in order, so it waits behind the tile that its other
// block is loading (see the tables in the kernel).
#include <type_traits>

#include "grid_tile.h"
#include "tile_math.h"

namespace moshpit {
namespace {

constexpr int kPositions = 8;                // of a group, per lane
constexpr int kRegisters = 8;                // of a thread for a table
constexpr int kAhead = 3;                    // rounds that the tables are read ahead
constexpr uint32_t kPlaceMask = 0x1fff1fffu; // a place has 13 bits; the other 3 of a lane's first two hold the group's count

// group of row `row` on axis `axis`
__device__ __forceinline__ int32_t group_of(const GridPlan &p, int32_t row, int32_t axis)
{
    const int32_t S = p.S[axis];
    const int32_t q = S == 1 ? row : quotient(row, p.magic_s[axis]);
    return quotient(q, p.magic_m) * S + (row - q * S);
}
__device__ __forceinline__ int32_t padded(const GridPlan &p, int32_t row)
{
    return row * p.part + (p.pad == 0 ? 0 : quotient(row, p.magic_m) * p.pad);
}
// LDS bytes of a peer's own row, and of the mean that round w of the pass writes for group g
__device__ __forceinline__ int32_t own_at(const GridPlan &p, int32_t row) { return padded(p, row); }
__device__ __forceinline__ int32_t mean_at(const GridPlan &p, int32_t w, int32_t g)
{
    return p.means_at + (w & 1) * p.means_bytes + padded(p, g);
}
// Where the entry of `row` stands in the table of final places: the rows of a thread next to each other.
__host__ __device__ __forceinline__ int32_t place_index(const GridPlan &p, int32_t row)
{
    const int32_t rows_per_slot = 64 >> p.wv_shift, per_wave = kPhaseSlots * p.phases * rows_per_slot;
    const int32_t in_wave = row % per_wave, slot = in_wave / rows_per_slot;
    const int32_t thread = (row / per_wave * rows_per_slot + in_wave % rows_per_slot) * p.phases + slot % p.phases;
    return thread * kPhaseSlots + slot / p.phases;
}
constexpr uint32_t kNoStore = 0xffffu;

typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) char lds_byte;
template <typename T> __device__ __forceinline__ T lds_get(uint32_t at)
{
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(at);
}
template <typename T> __device__ __forceinline__ void lds_put(uint32_t at, const T &v)
{
    *reinterpret_cast<__attribute__((address_space(3))) T *>(at) = v;
}

// 32-bit offset from a uniform address
template <typename T> __device__ __forceinline__ T table_get(const void *table, uint32_t at)
{
    return *reinterpret_cast<const T *>(static_cast<const char *>(table) + at);
}

// 16 * (lower or upper half of w) + col
template <int HALF> __device__ __forceinline__ uint32_t place(uint32_t w, uint32_t col)
{
    uint32_t a;
    if constexpr (HALF == 0) asm("v_mad_u32_u16 %0, %1, 16, %2" : "=v"(a) : "v"(w), "v"(col));
    else asm("v_mad_u32_u16 %0, %1, 16, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(w), "v"(col));
    return a;
}

// Tiles of two column parts come from memory with half the lanes of a wave holding one part, half the
// other.  exchange(a, b) of two slots leaves the first part of both in a and the second in b (lane of the
// lower half: of a's row, upper half: of b's), so that the registers of the part that is in LDS are free; it is its own
// inverse.  The halves are 32 lanes apart, or, where a row is a quad of lanes or less, 2 or 1.
template <int CTRL> __device__ __forceinline__ uint32_t quad_lane(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int DISTANCE> __device__ __forceinline__ void exchange(uint32_t &a, uint32_t &b)
{
    if constexpr (DISTANCE == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const uint32_t from_a = quad_lane<DISTANCE == 2 ? 0x4e : 0xb1>(a);
        const uint32_t from_b = quad_lane<DISTANCE == 2 ? 0x4e : 0xb1>(b);
        // (written out: as C++ selects they became branches with copies of every register)
        constexpr uint64_t kUpper = DISTANCE == 2 ? 0xccccccccccccccccull : 0xaaaaaaaaaaaaaaaaull;
        asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(a) : "v"(a), "v"(from_b), "s"(kUpper));
        asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(b) : "v"(from_a), "v"(b), "s"(kUpper));
    }
}
template <int DISTANCE> __device__ __forceinline__ void exchange_parts(u32x4 (&a)[kPhaseSlots], u32x4 (&b)[kPhaseSlots])
{
#pragma unroll
    for (int k = 0; k < kPhaseSlots; ++k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t lo = a[k][e], hi = b[k][e];
            exchange<DISTANCE>(lo, hi);
            a[k][e] = lo;
            b[k][e] = hi;
        }
    }
}

// SPLIT: lanes (16 or 32 apart) that share a group, 8 positions each.  HALF: 0 where the whole tile is in LDS; else
// its two column parts take turns, and HALF is the lanes between them in a wave that loads it.  NT: non-temporal loads and stores.  DIST: distortions are
// wanted.  TAB: where the places come from: kClosed (nobody is ever absent), kLds, kBits or kAheadOnly (see below).
template <int DT, int SPLIT, int HALF, bool NT, bool DIST, int TAB>
__global__ __launch_bounds__(HALF == 0 ? 1024 : 512, 4) void mean_rounds_kernel(char *X, GridPlan p)
{
    constexpr int PHASES = HALF == 0 ? 1 : 2;
    constexpr int kSlots = kPhaseSlots * PHASES;
    constexpr int kEs = DT == 0 ? 4 : 2;
    constexpr int NE = 16 / kEs;                             // columns of a lane's 16 bytes
    constexpr int NC = NE / SPLIT;                           // columns whose mean a lane forms
    extern __shared__ __align__(16) char lds[];
    const uint32_t base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte *)lds));

    const int32_t tid = threadIdx.x, T = blockDim.x, lane = tid & 63;
    const int32_t full_shift = p.wv_shift, full_mask = (1 << full_shift) - 1;      // vectors per row of the tile,
    const int32_t wv_shift = full_shift - (PHASES == 2 ? 1 : 0), wv_mask = (1 << wv_shift) - 1;     // of the part in LDS
    const int32_t part = 16 << wv_shift;

    // In memory, slot b of this thread is vector `vec` of row first_row + b * rows_per_slot.  In LDS it takes 8 vectors
    // of each part: vector `vec & wv_mask` of the rows lds_row + k * lds_step.
    const int32_t rows_per_slot = 64 >> full_shift;
    const bool upper = (lane & HALF) != 0;
    int32_t vec = lane & full_mask, row_in_slot = lane >> full_shift;
    if (HALF == 32) {
        vec = (lane & wv_mask) + (upper ? wv_mask + 1 : 0);
        row_in_slot = (lane & 31) >> wv_shift;
    }
    const int32_t first_row = (tid >> 6) * kSlots * rows_per_slot + row_in_slot;
    const int32_t lds_row = first_row + (upper ? rows_per_slot : 0), lds_step = PHASES * rows_per_slot;
    const int64_t w = tile_of(p, blockIdx.x);
    const TileSpan cur = tile_span(p, w);
    const bool in_tile = vec * 16 < cur.seg;
    const int32_t vec_at = vec * 16 < cur.seg - 16 ? vec * 16 : cur.seg - 16;      // (the row's last vector ends with the row)
    // (a slot outside the tile: the first row's vector)
    auto slot_offset = [&](int32_t row, int64_t row_bytes) -> int64_t {
        return static_cast<int64_t>(row < p.N ? row : 0) * row_bytes + vec_at;
    };

    // The lane's item: a (group, vector) pair, the lanes of a group 64 / SPLIT apart.  (Without tables: its first.)
    constexpr int kLanes = 64 / SPLIT;
    const int32_t sub = lane / kLanes;
    const int32_t item0 = (tid >> 6) * kLanes + (lane & (kLanes - 1)), item_step = T / SPLIT;
    const int32_t items = p.groups << wv_shift;
    const uint32_t out_at = SPLIT == 1 ? 0 : SPLIT == 2 ? sub * 8 : ((sub & 1) * 2 + (sub >> 1)) * 4;

    // waves that take a distortion (see there), and the thread's first term of one
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = T >> 6;
    const int32_t sharers = TAB == kLds ? waves / 2 : p.sharers, halves = TAB == kLds || waves > 1 ? 2 : 1;
    [[maybe_unused]] const int32_t first_term = (tid - (wave >= sharers ? sharers * 64 : 0)) >> wv_shift;

    // Tables.  Loads in the rounds would wait for the tile that the compute unit's other block is loading (a compute
    // unit returns loads in order), so the block takes what it can into registers along with its tile: with
    // TAB == kLds 4 bytes of a round's places, moves and terms per thread and register (1024 peers and more than 64
    // bytes of a row fill the threads once or less), `per_register` rounds in each of kRegisters.  Every round the threads that
    // hold them write those of the round after next to LDS, and the lanes read the next one's from there.  Where a row is
    // shorter a round's places would fill many registers.  There they come from two bits a position (kBits: does it
    // take part, was it averaged in the round before; 16 x 16 x 16 x 262,144 bfloat16, 12
    // rounds: 2.09 -> 1.90 ms; as 16-bit places read in the rounds 2.10, and with quotients by multiplication in place of the shifts 2.09), or, for
    // what bits cannot say (the donor of a returning peer) and with distortions, are loaded kAhead rounds ahead.
    const int32_t words_shift = p.words_shift, words = 1 << words_shift;      // of a round's places, two in each
    const int32_t per_register = T >> words_shift;           // (both are powers of two where there are tables)
    [[maybe_unused]] const int32_t per_shift = 31 - __builtin_clz(per_register > 0 ? per_register : 1);
    const int32_t move_words_max = words >> 1;                // of a round's moves; more are read from memory
    [[maybe_unused]] u32x8 entry_words, term_words;
    [[maybe_unused]] u32x4 move_words;
    u32x4 entry[TAB == kAheadOnly ? kAhead : 1];              // of the next round (kAheadOnly: rounds)
    uint32_t move[TAB == kAheadOnly ? kAhead : 1][2];
    [[maybe_unused]] uint32_t term[TAB == kAheadOnly ? kAhead : 1];
    // lane r: of round r
    int32_t moves = 0;
    [[maybe_unused]] int32_t terms = 0;
    [[maybe_unused]] uint32_t term0 = 0;
    u32x4 places{};
    auto fetch_round = [&](int i, int32_t ahead) {
        if constexpr (TAB == kAheadOnly) {
            const int64_t r = ahead < p.rounds ? ahead : ahead % p.rounds;
            const int32_t last = p.N << wv_shift;
            entry[i] = table_get<u32x4>(p.entries + r * p.groups * SPLIT * 4,
                                        static_cast<uint32_t>(item0 < items ? (item0 >> wv_shift) * SPLIT + sub : 0) * 16u);
#pragma unroll
            for (int k = 0; k < 2; ++k)
                move[i][k] = table_get<uint32_t>(p.moves + r * p.N, static_cast<uint32_t>((tid + k * T < last ? tid + k * T : 0) >> wv_shift) * 4u);
            if constexpr (DIST)
                term[i] = table_get<uint32_t>(p.terms + r * (p.N + p.groups), static_cast<uint32_t>(first_term < p.N ? first_term : 0) * 4u);
        }
    };
    // kBits: a group's bits in one word, a round's in T / groups threads; rows that move two to a thread and round, in
    // 24 bits (12 of the first and 4 of the second in row_words, two rounds to a word; 8 in row_bytes_4, four).
    constexpr int kRowRounds = 2 * kRegisters;
    [[maybe_unused]] u32x8 bit_words, row_words;
    [[maybe_unused]] u32x4 row_bytes_4;
    [[maybe_unused]] uint32_t group_bits = 0;
    const int32_t bit_threads = p.groups, bit_rounds = TAB == kBits ? T / bit_threads : 1;
    const int32_t bit_round = TAB == kBits ? tid / bit_threads : 0, bit_group = tid - bit_round * bit_threads;
    auto fetch_bits = [&](int32_t first) {
        if constexpr (TAB == kBits)
#pragma unroll
            for (int q = 0; q < kRegisters; ++q) {
                const int32_t r = first + q * bit_rounds + bit_round;
                bit_words[q] = table_get<uint32_t>(p.entries, static_cast<uint32_t>((r < p.rounds ? r : 0) * bit_threads + bit_group) * 4u);
            }
    };
    auto fetch_rows = [&](int32_t first) {                    // (the tables hold whole multiples of kRowRounds)
        if constexpr (TAB == kBits) {
#pragma unroll
            for (int q = 0; q < kRegisters; ++q) row_words[q] = table_get<uint32_t>(p.move_rows, static_cast<uint32_t>((first / 2 + q) * T + tid) * 4u);
#pragma unroll
            for (int q = 0; q < kRegisters / 2; ++q) row_bytes_4[q] = table_get<uint32_t>(p.move_bytes, static_cast<uint32_t>((first / 4 + q) * T + tid) * 4u);
        }
    };
    auto write_bits = [&](int32_t r) {
        if constexpr (TAB == kBits) {
            const int32_t in = r % (kRegisters * bit_rounds), q = in / bit_rounds;
            if (r > 0 && in == 0) fetch_bits(r);
            if (bit_round == in - q * bit_rounds) lds_put(base + p.words_at + (r & 1) * 4 * bit_threads + bit_group * 4, static_cast<uint32_t>(bit_words[q]));
        }
    };
    auto read_bits = [&](int32_t r) {
        if constexpr (TAB == kBits) group_bits = lds_get<uint32_t>(base + p.words_at + (r & 1) * 4 * bit_threads + (item0 < items ? item0 >> wv_shift : 0) * 4);
    };
    // kLds: rounds first .. first + kRegisters * per_register - 1 into the registers
    auto fetch_words = [&](int32_t first) {
        if constexpr (TAB == kLds) {
#pragma unroll
            for (int q = 0; q < kRegisters; ++q) {
                const int32_t r = first + q * per_register + (tid >> words_shift), word = tid & (words - 1);
                const bool there = r < p.rounds;
                const int64_t row = there ? r : 0;
                entry_words[q] = p.entries[row * words + word];
            }
#pragma unroll
            for (int q = 0; q < kRegisters / 2; ++q) {
                const int32_t r = first + q * 2 * per_register + (tid >> (words_shift - 1));
                move_words[q] = p.moves[static_cast<int64_t>(r < p.rounds ? r : 0) * p.N + (tid & (move_words_max - 1))];
            }
        }
    };
    [[maybe_unused]] auto fetch_terms = [&](int32_t first) {
        if constexpr (TAB == kLds && DIST)
#pragma unroll
            for (int q = 0; q < kRegisters; ++q) {
                const int32_t r = first + q * per_register + (tid >> words_shift);
                term_words[q] = p.terms[static_cast<int64_t>(r < p.rounds ? r : 0) * (p.N + p.groups) + (tid & (words - 1))];
            }
    };
    // kLds: those of round r from the registers to LDS
    auto write_words = [&](int32_t r) {
        if constexpr (TAB == kLds) {
            // (Quotients where the binary32 tile of 32 x 32 has two parts: slower by the divisions, its two blocks a compute unit fall into step less
            // often.  us, quotients : shifts, 8 rounds, 20 % absent: 4,194,304 elements 8,110 : 8,650, on one of six states
            // 9,060 : 8,970, 4,190,208 7,630 : 8,300, 3,145,728 7,510 : 7,370, 2,097,152 4,010 : 3,910, 6 rounds 3,930 : 4,020; 16 rounds
            // 12,750 : 12,280 and 6,800 : 6,580.  All other kernels, 60 MB to 17 GB, 8 and 16 rounds: shifts 0 to 9 % ahead on 34 shapes,
            // 16 x 16 x 976,576, 16 rounds, 590 : 539; none behind.)
            constexpr bool kQuotients = DT == 0 && SPLIT == 4 && HALF != 0 && !DIST;
            const int32_t in = kQuotients ? r % (kRegisters * per_register) : r & (kRegisters * per_register - 1);
            const int32_t q = kQuotients ? in / per_register : in >> per_shift;
            if (r > 0 && in == 0) fetch_words(r);
            if (tid >> words_shift == in - q * per_register) {
                lds_put(base + p.words_at + (r & 1) * 4 * words + (tid & (words - 1)) * 4, static_cast<uint32_t>(entry_words[q]));
            }
            if (tid >> (words_shift - 1) == in - q / 2 * 2 * per_register)
                lds_put(base + p.words_at + 8 * words + (r & 1) * 2 * words + (tid & (move_words_max - 1)) * 4, static_cast<uint32_t>(move_words[q / 2]));
        }
    };
    // (of round r itself: they are read behind its barrier; where LDS has room for one round's only (p.dist_barrier), the next
    // round's are written behind a barrier of the distortion)
    const uint32_t terms_at = base + p.words_at + 12 * words, terms_step = p.dist_barrier ? 0 : 4 * words;
    [[maybe_unused]] auto write_terms = [&](int32_t r) {
        if constexpr (TAB == kLds && DIST) {
            const int32_t in = r & (kRegisters * per_register - 1), q = in >> per_shift;
            if (r > 0 && in == 0) fetch_terms(r);
            if (tid >> words_shift == (in & (per_register - 1)))
                lds_put(terms_at + (r & 1) * terms_step + (tid & (words - 1)) * 4, static_cast<uint32_t>(term_words[q]));
        }
    };
    // kLds: the lane's own of round r from LDS
    auto read_words = [&](int32_t r) {
        if constexpr (TAB == kLds) {
            const uint32_t at = base + p.words_at + (r & 1) * 4 * words;
            entry[0] = lds_get<u32x4>(at + (item0 < items ? (item0 >> wv_shift) * SPLIT + sub : 0) * 16);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int32_t q = (tid + k * T) >> wv_shift;
                move[0][k] = lds_get<uint32_t>(base + p.words_at + 8 * words + (r & 1) * 2 * words + (q < move_words_max ? q : 0) * 4);
            }
        }
    };
    if (TAB != kClosed && p.rounds > 0) {
        // (before the tile's own loads, which they would wait for)
        const int32_t r = lane < p.rounds ? lane : 0;
        if constexpr (TAB == kAheadOnly)
#pragma unroll
            for (int i = 0; i < kAhead; ++i) fetch_round(i, i);
        fetch_words(0);
        fetch_terms(0);
        fetch_bits(0);
        fetch_rows(0);
        places = table_get<u32x4>(p.places, static_cast<uint32_t>(((tid >> 6) * rows_per_slot + row_in_slot) * PHASES + (upper ? 1 : 0)) * 16u);
        moves = p.move_counts[r];
        if constexpr (DIST) {
            terms = p.term_counts[r];
            term0 = p.terms[static_cast<int64_t>(r) * (p.N + p.groups)];
        }
    }

    u32x4 kept[PHASES][kPhaseSlots];
    {
        u32x4 pre[kSlots];
        const char *origin = X + cur.col0;
        int32_t row_ = first_row;
        asm volatile("" : "+v"(row_));               // keeps the address arithmetic out of registers that live across the rounds
#pragma unroll
        for (int b = 0; b < kSlots; ++b) {
            pre[b] = load_vec<NT, u32x4>(origin + slot_offset(row_ + b * rows_per_slot, p.row_bytes));
            if (PHASES == 2 && b % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // (few addresses at a time)
        }
#pragma unroll
        for (int k = 0; k < kSlots; ++k) kept[k % PHASES][k / PHASES] = pre[k];
        if constexpr (PHASES == 2) exchange_parts<HALF>(kept[0], kept[1]);
    }
    if constexpr (TAB != kClosed)
        for (int32_t q = tid; q <= kPositions * SPLIT; q += T) lds_put(base + p.rcp_at + q * 4, q == 0 ? 0.f : 1.f / static_cast<float>(q));
    if (tid <= wv_mask) lds_put(base + p.zero_at + tid * 16, u32x4{0u, 0u, 0u, 0u});

    // Mean of one group over 16 bytes (vector v): places of the 8 positions -> mean, written to dst.
    auto average = [&](const uint32_t (&at)[kPositions], uint32_t dst, float count, float y) {
        // kBatch positions are requested at once (few registers are free next to a second part of the tile)
        constexpr int kBatch = PHASES == 1 ? kPositions : kPositions / 2;
        constexpr int kIn = 4 / kEs;
        float f[NE];                             // sums of the positions
#pragma unroll
        for (int u0 = 0; u0 < kPositions; u0 += kBatch) {
            u32x4 raw[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) raw[u] = lds_get<u32x4>(at[u0 + u]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {        // 4 bytes of each at a time
                float x[kBatch][kIn];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if constexpr (DT == 0) {
                        x[u][0] = __uint_as_float(raw[u][q]);
                    } else {
                        x[u][0] = __uint_as_float(raw[u][q] << 16);
                        x[u][1] = __uint_as_float(raw[u][q] & 0xffff0000u);
                    }
                }
#pragma unroll
                for (int s = 1; s < kBatch; s *= 2)
#pragma unroll
                    for (int u = 0; u + s < kBatch; u += 2 * s)
#pragma unroll
                        for (int e = 0; e < kIn; ++e) x[u][e] += x[u + s][e];
#pragma unroll
                for (int e = 0; e < kIn; ++e) f[kIn * q + e] = u0 == 0 ? x[0][e] : f[kIn * q + e] + x[0][e];
                if constexpr (DT == 1) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (PHASES == 2) __builtin_amdgcn_sched_barrier(0);
        }
        float acc[NC];
        if constexpr (SPLIT == 1) {
#pragma unroll
            for (int e = 0; e < NC; ++e) acc[e] = 0.f + f[e];
        } else if constexpr (SPLIT == 2) {
#pragma unroll
            for (int e = 0; e < NC; ++e) {
                const LanePair a = swap32(f[e], f[e + NC]);      // lower half: column e, upper: e + NC
                acc[e] = 0.f + (a.first + a.second);
            }
        } else {
            float h[2 * NC];
#pragma unroll
            for (int e = 0; e < 2 * NC; ++e) {
                const LanePair a = swap16(f[e], f[e + 2 * NC]);  // rows 0, 2: column e; rows 1, 3: e + 2 NC
                h[e] = a.first + a.second;
            }
#pragma unroll
            for (int e = 0; e < NC; ++e) {
                const LanePair a = swap32(h[e], h[e + NC]);            // upper half: NC columns further
                acc[e] = 0.f + (a.first + a.second);
            }
        }
        divide_columns<NC>(acc, count, y);
        constexpr int kWords = NC * kEs / 4;
        uint32_t word[kWords];
#pragma unroll
        for (int k = 0; k < kWords; ++k) {
            if constexpr (DT == 0) word[k] = __float_as_uint(acc[k]);
            else word[k] = bf16_pair(acc[2 * k], acc[2 * k + 1]);
        }
        if constexpr (kWords == 4) lds_put(dst, u32x4{word[0], word[1], word[2], word[3]});
        else if constexpr (kWords == 2) lds_put(dst, u32x2{word[0], word[1]});
        else lds_put(dst, word[0]);
    };

    const float full_count = static_cast<float>(p.M);
    const float full_y = 1.f / full_count;

    // Round r of the pass on axis `axis`, of the part in LDS (seg bytes wide); its tables are in entry[i], move[i].
    auto round = [&](int i, int32_t seg, int32_t r, int32_t axis) {
        if constexpr (TAB == kBits) {
            const uint32_t bits = group_bits;
            if (r > 0 && r % kRowRounds == 0) fetch_rows(r);
            const uint32_t row_word = row_words[r % kRowRounds / 2] >> (r % 2 * 16), row_byte = row_bytes_4[r % kRowRounds / 4] >> (r % 4 * 8);
            if (r + 1 < p.rounds) read_bits(r + 1);
            if (r + 2 < p.rounds) write_bits(r + 2);
            // (groups of 16 and 16 bytes of a row: every quotient is a shift)
            const int32_t here = 4 * axis, there = 4 * (axis == 0 ? p.d - 1 : axis - 1);
            const uint32_t means_before = base + p.means_at + ((r + 1) & 1) * p.means_bytes;
            const auto at_row = [&](uint32_t row) -> uint32_t { return row * 16 + (row >> 4) * p.pad; };
            const auto before = [&](uint32_t row) -> uint32_t {           // place of the mean that the last round gave a row
                return means_before + at_row((row >> (there + 4)) << there | (row & ((1u << there) - 1u)));
            };
            const uint32_t count = __popc(bits & 0xffffu);
            if (count != 0 && (item0 & wv_mask) * 16 < seg) {
                const uint32_t g = item0, first = sub * kPositions;
                const uint32_t row0 = (g >> here) << (here + 4) | (g & ((1u << here) - 1u));
                const int32_t own_step = axis == 0 ? 16 : p.S[axis] * 16 + p.pad_step[axis], mean_step = p.mean_step[axis];
                uint32_t own = base + at_row(row0) + __umul24(first, own_step);
                uint32_t mean = before(row0) + __umul24(first, mean_step);
                const int32_t live = static_cast<int32_t>(bits >> first), was = static_cast<int32_t>(bits >> (16 + first));
                const uint32_t zero = base + p.zero_at;
                uint32_t at[kPositions];
#pragma unroll
                for (int u = 0; u < kPositions; ++u) {
                    const uint32_t averaged_before = static_cast<uint32_t>(__builtin_amdgcn_sbfe(was, u, 1));
                    const uint32_t on = static_cast<uint32_t>(__builtin_amdgcn_sbfe(live, u, 1));
                    const uint32_t from = (averaged_before & mean) | (~averaged_before & own);
                    at[u] = (on & from) | (~on & zero);
                    own += own_step;
                    mean += mean_step;
                }
                const float y = lds_get<float>(base + p.rcp_at + count * 4);
                average(at, base + p.means_at + (r & 1) * p.means_bytes + at_row(g) + out_at, static_cast<float>(count), y);
            }
            const int32_t n = __builtin_amdgcn_readlane(moves, r);
            auto one_move = [&](uint32_t row) { lds_put(base + at_row(row), lds_get<u32x4>(before(row))); };
            if (tid < n) one_move(row_word & 0xfffu);
            if (tid + T < n) one_move(((row_word >> 12) & 0xfu) | (row_byte & 0xffu) << 4);
#pragma unroll 1
            for (int32_t it = tid + 2 * T; it < n; it += T) {
                const uint32_t pair = table_get<uint32_t>(p.moves + static_cast<int64_t>(r) * p.N, static_cast<uint32_t>(it) * 4u);
                lds_put(place<1>(pair, base), lds_get<u32x4>(place<0>(pair, base)));
            }
        } else if constexpr (TAB != kClosed) {
            const u32x4 ent = entry[i];
            const uint32_t mv[2] = {move[i][0], move[i][1]};
            const int32_t move_items = __builtin_amdgcn_readlane(moves, r) << wv_shift;
            if constexpr (!DIST) fetch_round(i, r + kAhead);      // (DIST: after the distortion has used term[i])
            if (r + 1 < p.rounds) read_words(r + 1);
            if (r + 2 < p.rounds) write_words(r + 2);
            write_terms(r);
            const int32_t v = item0 & wv_mask;
            const uint32_t count = ((ent.x >> 13) & 7u) | ((ent.x >> 29) << 3);
            if (item0 < items && count != 0 && v * 16 < seg) {
                const uint32_t col = base + v * 16;
                uint32_t at[kPositions];
#pragma unroll
                for (int u = 0; u < kPositions / 2; ++u) {
                    const uint32_t pair = u == 0 ? ent[u] & kPlaceMask : ent[u];
                    at[2 * u] = place<0>(pair, col);
                    at[2 * u + 1] = place<1>(pair, col);
                }
                const float y = lds_get<float>(base + p.rcp_at + count * 4);
                average(at, col + mean_at(p, r, item0 >> wv_shift) + out_at, static_cast<float>(count), y);
            }
            auto one_move = [&](int32_t it, uint32_t pair) {
                const uint32_t col = base + (it & wv_mask) * 16;
                lds_put(place<1>(pair, col), lds_get<u32x4>(place<0>(pair, col)));
            };
            // (kLds: what is in LDS)
            const int32_t at_hand = TAB == kLds && move_words_max << wv_shift < move_items ? move_words_max << wv_shift : move_items;
            if (tid < at_hand) one_move(tid, mv[0]);
            if (tid + T < at_hand) one_move(tid + T, mv[1]);
#pragma unroll 1
            for (int32_t it = tid < at_hand ? tid + (tid + T < at_hand ? 2 : 1) * T : tid; it < move_items; it += T)
                one_move(it, table_get<uint32_t>(p.moves + static_cast<int64_t>(r) * p.N, static_cast<uint32_t>(it >> wv_shift) * 4u));
        } else {
            const int32_t before = axis == 0 ? p.d - 1 : axis - 1;
            const int32_t step = r > 0 ? p.mean_step[axis] : axis == 0 ? part : p.S[axis] * part + p.pad_step[axis];
            for (int32_t it = item0; it < items; it += item_step) {
                const int32_t g = it >> wv_shift, v = it & wv_mask;
                if (v * 16 >= seg) continue;
                const int32_t S = p.S[axis];
                const int32_t row0 = axis == 0 ? g * p.M : g + quotient(g, p.magic_s[axis]) * S * (p.M - 1);
                const uint32_t col = base + v * 16;
                uint32_t from = col + static_cast<uint32_t>(r > 0 ? mean_at(p, r - 1, group_of(p, row0, before)) : own_at(p, row0));
                from += __mul24(sub * kPositions, step);
                uint32_t at[kPositions];
#pragma unroll
                for (int u = 0; u < kPositions; ++u) {
                    at[u] = sub * kPositions + u < p.M ? from : col + p.zero_at;
                    from += step;
                }
                average(at, col + mean_at(p, r, g) + out_at, full_count, full_y);
            }
        }
    };

    // Distortion of the part in LDS after round r of the pass (r = -1: before the first): sum over
    // its columns of s2 - s1^2 / N, s1 and s2 the sums of the differences from one peer's row and of their
    // squares in binary64 (the differences are exact).  There are far fewer terms than threads, so the halves of a
    // block take the rounds in turn (sharers of its waves a round): thread (k, vector c) of the half takes every
    // parts-th term.  What the waves of a half leave in LDS is put together by its first wave after the next round's barrier, when the
    // other half is busy with that round's.
    const int32_t columns = NE << wv_shift;
    double *red = reinterpret_cast<double *>(lds + p.red_offset), *totals = red + halves * sharers * (columns + 1);
    [[maybe_unused]] auto sums_of = [&](int32_t r) -> double * { return red + (halves == 2 ? (r + 1) & 1 : 0) * sharers * (columns + 1); };
    [[maybe_unused]] auto first_wave = [&](int32_t r) -> int32_t { return halves == 2 ? ((r + 1) & 1) * sharers : 0; };
    [[maybe_unused]] auto distortion = [&](int i, int32_t seg, int32_t r) {
        if constexpr (DIST) {
            const int32_t w0 = first_wave(r);
            if (wave < w0 || wave >= w0 + sharers) return;
            const int32_t c = tid & wv_mask, first = first_term, parts = sharers * 64 >> wv_shift;
            const int32_t early = c * 16 - (seg - 16);             // > 0: the row's last vector, first `early` bytes not its own
            // (their bits are cleared in every term, and in the row that is subtracted)
            u32x4 own;
#pragma unroll
            for (int k = 0; k < 4; ++k) own[k] = early >= 4 * k + 4 ? 0u : early > 4 * k ? 0xffff0000u : ~0u;
            const uint32_t col = base + c * 16;
            const int32_t n = r < 0 ? p.N : TAB != kClosed ? __builtin_amdgcn_readlane(terms, r) : p.groups;
            const uint32_t *list = p.terms + static_cast<int64_t>(r < 0 ? 0 : r) * (p.N + p.groups);
            auto term_at = [&](int32_t k, float &weight) -> uint32_t {       // k < n
                weight = 1.f;
                if (r < 0) return col + own_at(p, k);
                if constexpr (TAB != kClosed) {
                    uint32_t t;
                    if (TAB == kLds && k < words) t = lds_get<uint32_t>(terms_at + (r & 1) * terms_step + k * 4);
                    else if (TAB == kAheadOnly && k == first) t = term[i];
                    else t = table_get<uint32_t>(list, static_cast<uint32_t>(k) * 4u);
                    weight = static_cast<float>(t >> 16);
                    return place<0>(t, col);
                } else {
                    return col + mean_at(p, r, k);               // (all terms count the same: below)
                }
            };
            float x0[NE];
            uint32_t at0 = col + (r < 0 ? own_at(p, 0) : mean_at(p, r, 0));
            if constexpr (TAB != kClosed)
                if (r >= 0) at0 = place<0>(__builtin_amdgcn_readlane(term0, r), col);
            widen16<DT>(lds_get<u32x4>(at0) & own, x0);
            double s1[NE], s2 = 0.0;
#pragma unroll
            for (int e = 0; e < NE; ++e) s1[e] = 0.0;
            auto add_terms = [&](auto rows_at_once, int32_t k0) {
                    constexpr int kRows = decltype(rows_at_once)::value;      // requested before the first is used
                    u32x4 raw[kRows];
                    float weight[kRows];
                    uint32_t at[kRows];
#pragma unroll
                    for (int u = 0; u < kRows; ++u) {
                        const int32_t k = k0 + u * parts;
                        at[u] = term_at(k < n ? k : first, weight[u]);
                        if (k >= n) at[u] = at0;                  // (its difference is 0)
                    }
#pragma unroll
                    for (int u = 0; u < kRows; ++u) raw[u] = lds_get<u32x4>(at[u]);
#pragma unroll
                    for (int u = 0; u < kRows; ++u) {
                        float x[NE];
                        widen16<DT>(raw[u] & own, x);
                        [[maybe_unused]] const double wt = static_cast<double>(weight[u]);
                        double sq = TAB == kClosed ? s2 : 0.0;
#pragma unroll
                        for (int e = 0; e < NE; ++e) {
                            const double dlt = static_cast<double>(x[e]) - static_cast<double>(x0[e]);
                            s1[e] = TAB == kClosed ? s1[e] + dlt : fma(wt, dlt, s1[e]);
                            sq = fma(dlt, dlt, sq);
                        }
                        s2 = TAB == kClosed ? sq : fma(wt, sq, s2);
                    }
            };
            if (c * 16 < seg && first < n) {
                // (most often there are fewer terms than threads for them)
                constexpr int kMany = PHASES == 1 ? 4 : 2;
                if (r < 0) {
                    for (int32_t k0 = first; k0 < n; k0 += kMany * parts) add_terms(std::integral_constant<int, kMany>(), k0);
                } else if (n <= parts) {
                    add_terms(std::integral_constant<int, 1>(), first);
                } else {
                    for (int32_t k0 = first; k0 < n; k0 += 2 * parts) add_terms(std::integral_constant<int, 2>(), k0);
                }
            }
            if (TAB == kClosed && r >= 0) {
                const double wt = static_cast<double>(full_count);
#pragma unroll
                for (int e = 0; e < NE; ++e) s1[e] *= wt;
                s2 *= wt;
            }
            double *sums = sums_of(r);
            column_sums<NE>(s1, s2, wv_shift, sums + (wave - w0) * columns, sums + sharers * columns + (wave - w0));
        }
    };
    // Behind the next barrier: the total of the distortion after round r.
    [[maybe_unused]] auto finish = [&](int32_t r) {
        if constexpr (DIST) {
            if (wave != first_wave(r) || !(r < 0 ? p.dist_before != 0 : ((p.dist_after >> r) & 1u) != 0)) return;
            const double sum = finish_columns(sums_of(r), sharers, columns, sums_of(r) + sharers * columns, sharers, p.peers, p.inv_n);
            if (lane == 0) totals[r + 1] = sum;
        }
    };
    // All totals of a part (its tile and number: part_at) leave LDS.
    [[maybe_unused]] auto write_distortions = [&](int64_t part_at) {
        if constexpr (DIST) {
            lds_barrier();
            finish(p.rounds - 1);
            lds_barrier();
            for (int32_t e = tid; e <= p.rounds; e += T)
                if (e == 0 ? p.dist_before != 0 : ((p.dist_after >> (e - 1)) & 1u) != 0) p.partials[e * p.tiles * PHASES + part_at] = totals[e];
        }
    };

    // Where the value of this thread's k-th row ends, in 16 bytes of LDS (column 0 of the part); kNoStore: it is not written back.
    const int32_t last_axis = (p.axis0 + p.rounds + p.d - 1) % p.d;
    auto final_at = [&](int k, int32_t row) -> uint32_t {
        if constexpr (TAB != kClosed) {
            const uint32_t word = places[k / 2];
            return k % 2 ? word >> 16 : word & 0xffffu;
        } else {
            return static_cast<uint32_t>(mean_at(p, p.rounds - 1, group_of(p, row, last_axis))) >> 4;
        }
    };
    uint32_t stored = 0;                                     // bit k: the k-th row is written back

#pragma unroll
    for (int32_t phase = 0; phase < PHASES; ++phase) {
        // bytes of this part
        const int32_t left = cur.seg - phase * part;
        const int32_t seg = left < part ? left : part;
        const int64_t tiles = p.tiles * PHASES;
        if (seg <= 0) {
            if constexpr (DIST)
                for (int32_t e = tid; e <= p.rounds; e += T)
                    if (e > 0 || p.dist_before) p.partials[e * tiles + w * PHASES + phase] = 0.0;
            break;
        }
        const bool mine = (vec & wv_mask) * 16 < seg;
        if (TAB == kAheadOnly && phase == 1) {
            // round r is in slot (p.rounds + r) % kAhead
            for (int32_t q = p.rounds % kAhead; q > 0; --q) {
                const u32x4 e = entry[0];
                const uint32_t m[2] = {move[0][0], move[0][1]};
                [[maybe_unused]] const uint32_t t = term[0];
                constexpr int kLast = TAB == kAheadOnly ? kAhead - 1 : 0;
#pragma unroll
                for (int i = 0; i < kLast; ++i) {
                    entry[i] = entry[i + 1];
                    move[i][0] = move[i + 1][0];
                    move[i][1] = move[i + 1][1];
                    if constexpr (DIST) term[i] = term[i + 1];
                }
                entry[kLast] = e;
                move[kLast][0] = m[0];
                move[kLast][1] = m[1];
                if constexpr (DIST) term[kLast] = t;
            }
        }
        if (TAB == kBits && p.rounds > 0) {
            if (phase == 1 && p.rounds > kRegisters * bit_rounds) fetch_bits(0);
            if (phase == 1 && p.rounds > kRowRounds) fetch_rows(0);
            write_bits(0);
            if (p.rounds > 1) write_bits(1);
        }
        if (TAB == kLds && p.rounds > 0) {
            // (the words of the first part's rounds have been read; they are still in the registers in a short run)
            if (phase == 1 && p.rounds > kRegisters * per_register) {
                fetch_words(0);
                fetch_terms(0);
            }
            write_words(0);
            if (p.rounds > 1) write_words(1);
        }
        int32_t row_ = lds_row;
        asm volatile("" : "+v"(row_));
#pragma unroll
        for (int k = 0; k < kPhaseSlots; ++k) {
            const int32_t row = row_ + k * lds_step;
            if (mine && row < p.N) lds_put(base + own_at(p, row) + (vec & wv_mask) * 16, kept[phase][k]);
        }
        lds_barrier();
        if (p.rounds > 0) {
            read_words(0);
            read_bits(0);
            // (the first round writes the third's over what is read here; later ones read a barrier before they are written over)
            if constexpr (TAB == kLds || TAB == kBits) lds_barrier();
        }

        if constexpr (DIST)
            if (p.dist_before) {
                distortion(0, seg, -1);
                if (p.dist_barrier) lds_barrier();
            }
        int32_t axis = p.axis0;
        constexpr int kUnroll = TAB == kAheadOnly ? kAhead : 1;            // (registers have no index)
#pragma unroll 1
        for (int32_t r0 = 0; r0 < p.rounds; r0 += kUnroll)
#pragma unroll
            for (int i = 0; i < kUnroll; ++i) {
                const int32_t r = r0 + i;
                if (r >= p.rounds) break;
                round(i, seg, r, axis);
                lds_barrier();
                if constexpr (DIST) {
                    finish(r - 1);
                    if ((p.dist_after >> r) & 1u) distortion(i, seg, r);
                    fetch_round(i, r + kAhead);
                    // (a returning peer may copy its donor to its own row, which the distortion has read)
                    if (p.dist_barrier) lds_barrier();
                }
                axis = axis + 1 == p.d ? 0 : axis + 1;
            }
        write_distortions(w * PHASES + phase);
        // back into the registers; the next part enters LDS when everybody is done with this one
        // (always read, whoever is stored, so that the registers need not keep what they held before)
        row_ = lds_row;
        asm volatile("" : "+v"(row_));
        stored = 0;
#pragma unroll
        for (int k = 0; k < kPhaseSlots; ++k) {
            const int32_t row = row_ + k * lds_step;
            const uint32_t at = row < p.N ? final_at(k, row) : kNoStore;
            stored |= (at != kNoStore ? 1u : 0u) << k;
            kept[phase][k] = lds_get<u32x4>(base + (at != kNoStore ? at : 0) * 16 + (vec & wv_mask) * 16);
        }
        if (PHASES == 2 && phase == 0) lds_barrier();
    }

    if (p.rounds > 0) {
        char *origin = X + cur.col0;
        int32_t row_ = first_row;
        asm volatile("" : "+v"(row_));
        uint32_t stored_upper = stored;
        if constexpr (PHASES == 2) {
            exchange_parts<HALF>(kept[0], kept[1]);
            const uint32_t mine = stored, other = static_cast<uint32_t>(__shfl_xor(static_cast<int>(stored), HALF, 64));
            stored = upper ? other : mine;
            stored_upper = upper ? mine : other;
        }
#pragma unroll
        for (int k = 0; k < kPhaseSlots; ++k) {
#pragma unroll
            for (int b = 0; b < PHASES; ++b)
                if (in_tile && (((b == 0 ? stored : stored_upper) >> k) & 1u))
                    store_vec<NT, u32x4>(origin + slot_offset(row_ + (PHASES * k + b) * rows_per_slot, p.row_bytes), kept[b][k]);
            if (PHASES == 2 && k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// ---- the tables: one launch per run --------------------------------------------------------------

// Ranks of the set flags among those of the block, in the order of k * kPlanThreads + thread; returns how many there are.
__device__ __forceinline__ int32_t block_ranks(const bool (&flag)[kPerThread], int32_t (&rank)[kPerThread], int32_t *sums)
{
    constexpr int kWaves = kPlanThreads / 64;
    static_assert(kPerThread * kWaves == 64, "one sum per lane");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long ballot[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        ballot[k] = __ballot(flag[k]);
        if (lane == 0) sums[k * kWaves + wave] = __popcll(ballot[k]);
    }
    __syncthreads();
    int32_t up_to = sums[lane];
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t before = __shfl_up(up_to, off, 64);
        if (lane >= off) up_to += before;
    }
    const int32_t total = __shfl(up_to, 63, 64);
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t at = k * kWaves + wave;
        const int32_t below = at == 0 ? 0 : __shfl(up_to, at - 1, 64);
        rank[k] = below + __popcll(ballot[k] & ((1ull << lane) - 1ull));
    }
    __syncthreads();
    return total;
}

__device__ __forceinline__ bool present_in(const GridSchedule &s, int32_t i, int64_t r)
{
    return s.masks != nullptr ? s.masks[r * s.N + i] != 0 : !failure_event(s.seed, s.t0 + r, i, s.threshold);
}

// Participants of a group, or 0 where nobody is averaged.
__device__ __forceinline__ uint32_t averaged(const GridSchedule &s, uint32_t bits)
{
    const int32_t n = __popc(bits);
    return n < 2 || (s.group_skip && n != s.M) ? 0u : bits;
}

// place of row `row` within its group on axis `axis`
__device__ __forceinline__ int32_t position_of(const GridPlan &p, int32_t row, int32_t axis)
{
    const int32_t q = p.S[axis] == 1 ? row : quotient(row, p.magic_s[axis]);
    return q - quotient(q, p.magic_m) * p.M;
}

__device__ __forceinline__ int32_t plan_axis(const GridSchedule &s, int64_t r) { return static_cast<int32_t>((s.t0 + r) % s.d); }

// Where peer i's value stands after the last round of its pass, if it took part in the pass.
__device__ __forceinline__ void write_place(const GridSchedule &s, const GridPlan &p, const MeanTables &o, int32_t pass, int32_t i,
                                            bool took_part, bool averaged_last)
{
    const int32_t first = pass * o.pass_rounds, end = first + o.pass_rounds < s.rounds ? first + o.pass_rounds : s.rounds;
    uint32_t at = kNoStore;
    if (took_part)
        at = static_cast<uint32_t>(averaged_last ? mean_at(p, end - 1 - first, group_of(p, i, plan_axis(s, end - 1))) : own_at(p, i)) >> 4;
    o.places[static_cast<int64_t>(pass) * o.place_stride + place_index(p, i)] = static_cast<uint16_t>(at);
}

// Blocks 0 .. rounds-1: round r = blockIdx.x of the tables (entries, moves, terms).  Blocks
// after that, one for each pass: the final places; under group-skip schedules those come from mean_places_kernel.
__global__ __launch_bounds__(kPlanThreads) void mean_plan_kernel(GridSchedule s, GridPlan p, MeanTables o)
{
    __shared__ uint16_t source[kGridMaxPeers];                // where a peer's value is, in 16 bytes of LDS
    __shared__ uint16_t candidates[kGridMaxPeers];
    __shared__ uint32_t bits_now[kGridMaxPeers / 2], bits_before[kGridMaxPeers / 2];
    __shared__ uint32_t o_rows[kPlanThreads];                 // plan.bits: the two rows that a thread moves, 12 bits each
    __shared__ int32_t sums[64];
    const int32_t N = s.N, M = s.M, groups = N / M, tid = threadIdx.x;
    if (static_cast<int32_t>(blockIdx.x) >= s.rounds) {
        const int32_t pass = static_cast<int32_t>(blockIdx.x) - s.rounds;
        const int32_t first = pass * o.pass_rounds, end = first + o.pass_rounds < s.rounds ? first + o.pass_rounds : s.rounds;
        const int32_t axis = plan_axis(s, end - 1);
        for (int32_t g = tid; g < groups; g += kPlanThreads) bits_now[g] = 0;
        __syncthreads();
        bool last[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int32_t i = tid + k * kPlanThreads;
            last[k] = i < N && present_in(s, i, end - 1);
            if (last[k]) atomicOr(&bits_now[group_of(p, i, axis)], 1u << position_of(p, i, axis));
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int32_t i = tid + k * kPlanThreads;
            if (i >= N) continue;
            bool took_part = last[k];
            for (int32_t r = end - 2; r >= first && !took_part; --r) took_part = present_in(s, i, r);
            write_place(s, p, o, pass, i, took_part, last[k] && averaged(s, bits_now[group_of(p, i, axis)]) != 0);
        }
        return;
    }
    const int32_t r = blockIdx.x, within = r % o.pass_rounds;
    const int32_t axis = plan_axis(s, r), before = axis == 0 ? s.d - 1 : axis - 1;
    const bool refresh = s.refresh && (r > 0 || s.continued);
    const bool follows = within > 0;                          // the pass has a round before this one
    bool was[kPerThread], is[kPerThread];
    for (int32_t g = tid; g < groups; g += kPlanThreads) bits_now[g] = bits_before[g] = 0;
    o_rows[tid] = 0;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        is[k] = i < N && present_in(s, i, r);
        was[k] = i < N && (follows || refresh) && present_in(s, i, r - 1);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        if (is[k]) atomicOr(&bits_now[group_of(p, i, axis)], 1u << position_of(p, i, axis));
        if (follows && was[k]) atomicOr(&bits_before[group_of(p, i, before)], 1u << position_of(p, i, before));
    }
    __syncthreads();
    for (int32_t g = tid; g < groups; g += kPlanThreads) {
        bits_now[g] = averaged(s, bits_now[g]);
        bits_before[g] = averaged(s, bits_before[g]);
        if (o.bitmaps != nullptr) o.bitmaps[static_cast<int64_t>(r) * groups + g] = bits_now[g];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        if (i >= N) continue;
        const int32_t g = group_of(p, i, before);
        const bool moved = follows && was[k] && bits_before[g] != 0;
        source[i] = static_cast<uint16_t>((moved ? mean_at(p, within - 1, g) : own_at(p, i)) >> 4);
    }
    if (refresh) {
        // returning peers read their donors' rows (who do not return themselves)
        bool flag[kPerThread];
        int32_t rank[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) flag[k] = was[k] && is[k];
        const int32_t c = block_ranks(flag, rank, sums);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)
            if (flag[k]) candidates[rank[k]] = static_cast<uint16_t>(tid + k * kPlanThreads);
        __syncthreads();
        const uint64_t round_key = mix64(s.seed + 0xA0761D6478BD642Full * static_cast<uint64_t>(s.t0 + r + 1));
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int32_t i = tid + k * kPlanThreads;
            if (c > 0 && is[k] && !was[k]) {
                const uint64_t u = mix64(round_key ^ static_cast<uint64_t>(i));
                source[i] = source[candidates[u % static_cast<uint64_t>(c)]];
            }
        }
    }
    __syncthreads();
    const int32_t width = kPositions * p.split;
    uint16_t *entries = reinterpret_cast<uint16_t *>(o.entries) + static_cast<int64_t>(r) * groups * width;
    if (p.bits)
        for (int32_t g = tid; g < groups; g += kPlanThreads) {
            // (who was averaged in the round before, by this round's groups)
            uint32_t was_bits = 0;
            for (int32_t j = 0; j < M; ++j) {
                const int32_t i = g / p.S[axis] * p.S[axis] * M + g % p.S[axis] + j * p.S[axis];
                was_bits |= static_cast<uint32_t>(source[i] != static_cast<uint16_t>(own_at(p, i) >> 4)) << j;
            }
            o.entries[static_cast<int64_t>(r) * groups + g] = bits_now[g] | was_bits << 16;
        }
    for (int32_t q = tid; !p.bits && q < groups * width; q += kPlanThreads) {
        const int32_t g = q / width, j = q % width, S = p.S[axis];
        const bool on = (bits_now[g] >> j) & 1u;              // (positions past the group are never set)
        const uint32_t at = on ? source[g / S * S * M + g % S + j * S] : static_cast<uint32_t>(p.zero_at) >> 4;
        const uint32_t count = __popc(bits_now[g]);
        const uint32_t extra = j % kPositions == 0 ? count & 7u : j % kPositions == 1 ? count >> 3 : 0u;
        entries[q] = static_cast<uint16_t>(at | extra << 13);
    }
    // Peers that this round passes over: their value goes back to their own row, and they are terms of their own.
    bool rest[kPerThread], moves[kPerThread];
    int32_t rank[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        rest[k] = i < N && !(is[k] && bits_now[group_of(p, i, axis)] != 0);
        moves[k] = rest[k] && source[i < N ? i : 0] != static_cast<uint16_t>(own_at(p, i) >> 4);
    }
    const int32_t n_moves = block_ranks(moves, rank, sums);
    if (tid == 0) o.move_counts[r] = n_moves;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        if (!moves[k]) continue;
        o.moves[static_cast<int64_t>(r) * N + rank[k]] = source[i] | static_cast<uint32_t>(own_at(p, i) >> 4) << 16;
        if (p.bits && rank[k] < 2 * p.threads) atomicOr(&o_rows[rank[k] % p.threads], static_cast<uint32_t>(i) << (rank[k] / p.threads * 12));
    }
    if (p.bits) {
        __syncthreads();
        for (int32_t t = tid; t < p.threads; t += kPlanThreads) {
            reinterpret_cast<uint16_t *>(o.move_rows)[2 * (static_cast<int64_t>(r / 2) * p.threads + t) + r % 2] = static_cast<uint16_t>(o_rows[t] & 0xffffu);
            reinterpret_cast<uint8_t *>(o.move_bytes)[4 * (static_cast<int64_t>(r / 4) * p.threads + t) + r % 4] = static_cast<uint8_t>(o_rows[t] >> 16);
        }
    }
    if (o.terms == nullptr) return;
    uint32_t *terms = o.terms + static_cast<int64_t>(r) * (N + groups);
    const int32_t n_rest = block_ranks(rest, rank, sums);
    if (tid == 0) o.term_counts[r] = groups + n_rest;
    for (int32_t g = tid; g < groups; g += kPlanThreads) {
        const uint32_t count = __popc(bits_now[g]);
        // (a group without an average: any row, with weight 0)
        terms[g] = static_cast<uint32_t>(count != 0 ? mean_at(p, within, g) : own_at(p, g / p.S[axis] * p.S[axis] * M + g % p.S[axis])) >> 4 | count << 16;
    }
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
        const int32_t i = tid + k * kPlanThreads;
        if (rest[k]) terms[groups + rank[k]] = static_cast<uint32_t>(own_at(p, i)) >> 4 | 1u << 16;
    }
}

// Final places under group-skip schedules: a peer whose groups all sit out is not touched,
// unless it is refreshed.
__global__ __launch_bounds__(256) void mean_places_kernel(GridSchedule s, GridPlan p, MeanTables o)
{
    const int32_t groups = s.N / s.M, per_pass = (s.N + 255) / 256;
    const int32_t pass = static_cast<int32_t>(blockIdx.x) / per_pass;
    const int32_t i = static_cast<int32_t>(blockIdx.x) % per_pass * 256 + threadIdx.x;
    if (i >= s.N) return;
    const auto in_average = [&](int32_t r) {
        const int32_t axis = plan_axis(s, r);
        return ((o.bitmaps[static_cast<int64_t>(r) * groups + group_of(p, i, axis)] >> position_of(p, i, axis)) & 1u) != 0;
    };
    const int32_t first = pass * o.pass_rounds, end = first + o.pass_rounds < s.rounds ? first + o.pass_rounds : s.rounds;
    bool took_part = false;
    for (int32_t r = first; r < end && !took_part; ++r)
        took_part = in_average(r) || (s.refresh && present_in(s, i, r));
    write_place(s, p, o, pass, i, took_part, in_average(end - 1));
}

}  // namespace

hipError_t launch_mean_plan(const GridSchedule &s, const GridPlan &plan, const MeanTables &tables, hipStream_t stream)
{
    if (s.rounds <= 0) return hipSuccess;
    const int32_t passes = (s.rounds + tables.pass_rounds - 1) / tables.pass_rounds;
    const int32_t place_blocks = s.group_skip ? 0 : passes;
    mean_plan_kernel<<<dim3(static_cast<uint32_t>(s.rounds + place_blocks)), dim3(kPlanThreads), 0, stream>>>(s, plan, tables);
    if (s.group_skip)
        mean_places_kernel<<<dim3(static_cast<uint32_t>(passes * ((s.N + 255) / 256))), dim3(256), 0, stream>>>(s, plan, tables);
    return hipGetLastError();
}

namespace {

typedef void (*mean_kernel_t)(char *, GridPlan);

template <int DT, int SPLIT, int HALF, int TAB, bool NT, bool DIST> mean_kernel_t built()
{
    if constexpr (mean_kernel_built(DT, SPLIT, HALF, NT, DIST, TAB)) return mean_rounds_kernel<DT, SPLIT, HALF, NT, DIST, TAB>;
    else return nullptr;
}
template <int DT, int SPLIT, int HALF, int TAB> mean_kernel_t pick_mode(const MeanKernel &k)
{
    return k.nt ? (k.dist ? built<DT, SPLIT, HALF, TAB, true, true>() : built<DT, SPLIT, HALF, TAB, true, false>())
                : (k.dist ? built<DT, SPLIT, HALF, TAB, false, true>() : built<DT, SPLIT, HALF, TAB, false, false>());
}
template <int DT, int SPLIT, int HALF> mean_kernel_t pick_tables(const MeanKernel &k)
{
    return k.tab == kClosed ? pick_mode<DT, SPLIT, HALF, kClosed>(k) : k.tab == kLds ? pick_mode<DT, SPLIT, HALF, kLds>(k)
         : k.tab == kAheadOnly ? pick_mode<DT, SPLIT, HALF, kAheadOnly>(k) : pick_mode<DT, SPLIT, HALF, kBits>(k);
}
template <int DT, int SPLIT> mean_kernel_t pick_parts(const MeanKernel &k)
{
    return k.half == 0 ? pick_tables<DT, SPLIT, 0>(k) : k.half == 1 ? pick_tables<DT, SPLIT, 1>(k)
         : k.half == 2 ? pick_tables<DT, SPLIT, 2>(k) : pick_tables<DT, SPLIT, 32>(k);
}
template <int DT> mean_kernel_t pick_kernel(const MeanKernel &k)
{
    return k.split == 1 ? pick_parts<DT, 1>(k) : k.split == 2 ? pick_parts<DT, 2>(k) : pick_parts<DT, 4>(k);
}

}  // namespace

hipError_t launch_mean_rounds(void *X, int dtype, const GridPlan &plan, hipStream_t stream)
{
    GridPlan p = plan;
    const bool dist = p.partials != nullptr;
    p.lds_bytes = static_cast<int32_t>(means_lds_bytes(p, p.entries != nullptr, p.rounds, dist, dtype == 0 ? 4 : 2, &p.red_offset));
    if (p.lds_bytes > kLdsPerBlock || p.tiles > 0x7fffffffLL || p.grad != nullptr) return hipErrorInvalidValue;
    const MeanKernel which = mean_kernel(p, p.entries != nullptr, dist);
    const mean_kernel_t kernel = dtype == 0 ? pick_kernel<0>(which) : pick_kernel<1>(which);
    if (kernel == nullptr) return hipErrorInvalidValue;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), kLdsPerBlock);
    if (e != hipSuccess) return e;
    kernel<<<dim3(static_cast<uint32_t>(p.tiles)), dim3(p.threads), p.lds_bytes, stream>>>(static_cast<char *>(X), p);
    return hipGetLastError();
}

}  // namespace moshpit
