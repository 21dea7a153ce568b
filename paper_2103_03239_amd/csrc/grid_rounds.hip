// Consecutive averaging rounds on a WHOLE grid of up to 4096 peers in one pass over HBM, for
// gfx950: the loop of Alg. 1 with everything a run may ask for in between - the distortion after
// every round (left-hand side of the equation of Thm 3.2), the refresh of returning peers (App.
// "Training with a dynamic number of peers") and the local step of Moshpit SGD (Alg. 2).
//
// Columns never interact (the convergence argument of App. C.2 is component-wise), so a tile made
// of ALL N rows and Wb bytes of each is closed under every one of these steps: it is read from HBM
// once, the rounds run on it in LDS, and it is written back once.  Values live in LDS in the
// storage type and a round uses the arithmetic of the single-round kernel (same balanced tree of
// 16-position blocks, one correctly rounded division, one rounding to the storage type), so the
// state after a pass has the bits of the same rounds run one by one.
//
// Tiles.  Wb is a power of two: as wide as 32 KiB of tile allow (1 KiB at most), 256 bytes up to
// 64 KiB, 128 bytes for up to 1024 peers, 64 for up to 2048 and 32 above.  A block holds its tile 16 bytes at a
// time in the registers of its threads and works on it in LDS, at most 64 KiB at once, so that two
// blocks or more share a compute unit: one block's loads and stores overlap another's rounds.  (A
// wave that issues vector memory instructions faster than its compute unit's share of HBM delivers
// is held at the issue; with one block of 128 KiB per compute unit that prefetched its next tile
// the memory time and the time of the rounds added up.)  Tiles of 128 KiB wait in the registers
// and pass through LDS in two column parts, so that HBM still sees the full width.  Next to 16 slots
// few of the 128 registers of a thread are free: the two-part kernels with the distortion keep 20 to 36
// bytes a lane in scratch (14 of the 80 kernels; the others none).
//
// What bounds it (MI355X).  Up to about 6 rounds the memory side: 64 rows of 102 MB in tiles of
// 512 bytes 5.1 TB/s, 256 rows of 4 MiB in tiles of 256 bytes 5.4 TB/s (a copy in that pattern
// gives 5.3 and 5.5); 1024 rows of 16 MiB in tiles of 128 bytes 4.2 TB/s (copy: 4.2 - 4.5).  Then
// LDS: a round reads and rewrites the tile, 35 us per GiB of state and round on 16 x 16 peers (the
// LDS of the chip reads a GiB in 14 us and writes it in 23 us).
// Measured against the persistent kernel of fused_rounds.hip, which serves the larger grids:
// 4 x 4 x 4 peers x 25,557,032 binary32, 6 rounds 2.92 -> 2.56 ms; 32 x 32 x 4,194,304, 8 rounds
// 10.6 -> 9.3 ms; 16 x 16 x 16 x 262,144 bfloat16, 12 rounds 5.15 -> 2.08 ms (one pass instead
// of six over planes of 256 rows; 32-byte rows move at 3.7 TB/s, see tile_of).  Longer runs of groups of more than 4
// are taken over by the kernel of mean_rounds.hip (choose_means in grid_plan.h).
//
// Row ends and alignment.  Rows need no alignment beyond the element's: the loads and stores are
// 128-bit accesses at element-aligned addresses.  Where a row does not end on a 16-byte boundary
// the tile's last vector starts early enough to end with the row; the columns it shares with its
// neighbour are averaged twice, with the same bits.
#include <type_traits>

#include "grid_tile.h"
#include "sum_partials.h"
#include "tile_math.h"

namespace moshpit {
namespace {

// TREE, SPLIT, PER as chosen from M: TREE = summation block (power of two >= M, at most 16);
// SPLIT lanes of a wave share the positions of a group, PER positions each (SPLIT = 1: one lane
// takes them all).  PHASES: column parts of the tile that take turns in LDS.  NT: non-temporal
// loads and stores.  DIST: distortions are wanted.
template <int DT, int TREE, int SPLIT, int PER, int PHASES, bool NT, bool DIST>
__global__ __launch_bounds__(PHASES == 1 ? 1024 : 512, 4) void grid_rounds_kernel(char *X, GridPlan p)
{
    constexpr int kSlots = kPhaseSlots * PHASES;
    constexpr int CV = 4;                                    // columns per item
    typedef Cols<DT, CV> Q;
    typedef typename Q::elem_t elem_t;
    typedef typename std::conditional<SPLIT == 4, uint32_t, uint16_t>::type bits_t;      // M <= 16 but for SPLIT == 4
    constexpr int kEs = sizeof(elem_t);
    constexpr int NE = 16 / kEs;
    constexpr int FLAT = 16 / CV;
    extern __shared__ __align__(16) char lds[];
    char *tile = lds;
    bits_t *bitmaps = reinterpret_cast<bits_t *>(lds + p.tile_bytes);
    uint8_t *flags = reinterpret_cast<uint8_t *>(bitmaps + p.rounds * p.groups);
    double *red = reinterpret_cast<double *>(lds + p.red_offset);      // DIST: [dist_sum_rows][columns], then [waves]
    float *rcp_tab = reinterpret_cast<float *>(lds + p.lds_bytes - 32 - kRcpBytes);
    elem_t *zeros = reinterpret_cast<elem_t *>(lds + p.lds_bytes - 32);
    elem_t *trash = reinterpret_cast<elem_t *>(lds + p.lds_bytes - 16);

    const int32_t tid = threadIdx.x, T = blockDim.x;
    // The tile has 2^full_shift vectors per row, the part of it that is in LDS 2^wv_shift.
    const int32_t full_shift = p.wv_shift, full_mask = (1 << full_shift) - 1;
    const int32_t wv_shift = full_shift - (PHASES == 2 ? 1 : 0), wv_mask = (1 << wv_shift) - 1;
    const int32_t Wb = 16 << wv_shift;               // bytes of a row in LDS

    // slot b of this thread: vector idx & full_mask of row idx >> full_shift, idx = tid + b * T
    u32x4 pre[kSlots];
    auto slot_valid = [&](const TileSpan &t, int32_t idx) -> bool {
        return (idx >> full_shift) < p.N && (idx & full_mask) * 16 < t.seg;
    };
    // where slot idx lives in a matrix whose rows are row_bytes apart (a slot outside the tile: its first vector)
    auto slot_offset = [&](const TileSpan &t, int32_t idx, int64_t row_bytes) -> int64_t {
        if (!slot_valid(t, idx)) idx = 0;
        const int32_t row = idx >> full_shift, v16 = (idx & full_mask) * 16;
        const int32_t last = t.seg - 16;
        return static_cast<int64_t>(row) * row_bytes + (v16 < last ? v16 : last);
    };
    // vector v of row `row` of the part in LDS
    auto lds_vec = [&](int32_t row, int32_t v) -> u32x4 * {
        const int32_t pad = p.pad == 0 ? 0 : quotient(row, p.magic_m) * p.pad;
        return reinterpret_cast<u32x4 *>(tile + row * Wb + v * 16 + pad);
    };
    auto fetch = [&](const TileSpan &t) {
        const char *origin = X + t.col0;
        int32_t t_ = tid;
        asm volatile("" : "+v"(t_));                 // keeps the address arithmetic out of registers that live across the rounds
#pragma unroll
        for (int b = 0; b < kSlots; ++b)
            pre[b] = load_vec<NT, u32x4>(origin + slot_offset(t, t_ + b * T, p.row_bytes));
    };

    const int64_t w = tile_of(p, blockIdx.x);
    const TileSpan cur = tile_span(p, w);
    fetch(cur);

    for (int32_t q = tid; q < p.rounds * p.groups; q += T) bitmaps[q] = static_cast<bits_t>(p.bitmaps != nullptr ? p.bitmaps[q] : p.full_bitmap);
    for (int32_t q = tid; q < p.N; q += T) flags[q] = p.flags != nullptr ? p.flags[q] : 3;
    if (tid < 4) reinterpret_cast<uint32_t *>(zeros)[tid] = 0u;
    for (int32_t q = tid; q <= 64; q += T) rcp_tab[q] = q == 0 ? 0.f : 1.f / static_cast<float>(q);
    if (p.grad != nullptr) lds_barrier();            // the local step reads the flags

    // One round on axis `axis`, with the participant bitmaps bm[], of the part in LDS (seg bytes wide).
    auto round = [&](int32_t seg, int32_t axis, const bits_t *bm) {
        const int32_t chunk_shift = wv_shift + (kEs == 4 ? 0 : 1);              // log2 of CV-column chunks per row
        const int32_t chunk_mask = (1 << chunk_shift) - 1;
        const int32_t seg16 = (seg + 15) & ~15;            // (the last vector fills its slot)
        const int32_t S = p.S[axis];
        const uint32_t magic_s = p.magic_s[axis];
        const int32_t step = axis == 0 ? Wb : S * Wb + p.pad_step[axis];    // bytes between the rows of a group
        constexpr int kLanes = 64 / SPLIT;
        const int32_t sub = (tid & 63) / kLanes;
        int32_t it = (tid >> 6) * kLanes + (tid & (kLanes - 1));
        const int32_t it_step = T / SPLIT;
        for (; it < (p.groups << chunk_shift); it += it_step) {
            const int32_t gl = it >> chunk_shift, cc = it & chunk_mask;
            const uint32_t live = bm[gl];
            const int cnt = __popc(live);
            if (cnt < 2 || cc * (CV * kEs) >= seg16) continue;
            [[maybe_unused]] float y = 0.f;
            if constexpr (SPLIT == 1) y = rcp_tab[cnt];
            const int32_t row0 = axis == 0 ? gl * p.M : gl + quotient(gl, magic_s) * S * (p.M - 1);
            int32_t at = row0 * Wb + cc * (CV * kEs);
            if (p.pad != 0) at += (axis == 0 ? gl : quotient(row0, p.magic_m)) * p.pad;
            char *col = tile + at;
            float acc[CV];
            if constexpr (SPLIT > 1) {
                int32_t st = step;
                asm volatile("" : "+s"(st));
                const int32_t j0 = sub * PER;
                const uint32_t pbits = (live >> j0) & ((1u << PER) - 1u);
                char *q = col + __mul24(j0, st);
                elem_t *pos[PER];
                float f[PER][CV];
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const bool on = (pbits >> u) & 1u;
                    elem_t *e = reinterpret_cast<elem_t *>(q);
                    Q::load(on ? e : zeros, f[u]);
                    pos[u] = on ? e : trash;
                    q += st;
                }
#pragma unroll
                for (int s = 1; s < PER; s *= 2)
#pragma unroll
                    for (int u = 0; u + s < PER; u += 2 * s)
#pragma unroll
                        for (int e = 0; e < CV; ++e) f[u][e] += f[u + s][e];
                mean_over_lanes<SPLIT>(f[0], static_cast<float>(cnt), acc);
#pragma unroll
                for (int u = 0; u < PER; ++u) Q::store(pos[u], acc);
            } else {
                elem_t *base = reinterpret_cast<elem_t *>(col);
                const int32_t estep = step / kEs;
                float sum[CV];
                tree_block<DT, CV, TREE, FLAT>(base, estep, 0, zeros, live, sum);
#pragma unroll
                for (int e = 0; e < CV; ++e) acc[e] = 0.f + sum[e];
                divide_columns<CV>(acc, static_cast<float>(cnt), y);
                if constexpr (TREE < 16) {
#pragma unroll
                    for (int u = 0; u < TREE; ++u)
                        if ((live >> u) & 1u) Q::store(base + u * estep, acc);
                } else {
#pragma unroll
                    for (int u = 0; u < TREE; ++u) Q::store(((live >> u) & 1u) ? base + u * estep : trash, acc);
                }
            }
        }
    };

    // Distortion of the tile: sum over its columns of s2 - s1^2 / N, s1 and s2 the sums of the
    // differences from row 0 and of their squares in binary64 (the differences are exact).  The lanes and waves that share a column
    // are added in a fixed order; what they left is put together by one wave behind the barrier that every distortion needs (the
    // next round writes over the rows), while the others go on.
    // Rows of 256 bytes and more: a thread takes 4 bytes of every parts-th row, so that a wave shares its columns with the waves of
    // other parts only, in wide tiles of few rows with nobody.  Shorter rows: 16 bytes, and the lanes that share a column are summed
    // by exchanges (column_sums).  Vector instructions bound it: 3 x 3 x 3 x 7,875,648 bfloat16, 9 distortions 1.26 -> 0.81 ms,
    // 4 x 4 x 6,643,636 binary32, 11 distortions 708 -> 577 us against 16 bytes everywhere with all lanes' sums through LDS.
    [[maybe_unused]] auto distortion = [&](int32_t seg, int32_t entry, int64_t out_at) {
        if constexpr (DIST) {
            const int32_t waves = T >> 6, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            int32_t columns = NE << wv_shift, parts = waves;
            double *squares = red + dist_sum_rows(T, Wb, PHASES) * columns;
            if (PHASES == 1 && wv_shift >= 4) {
                constexpr int kIn = 4 / kEs;
                const int32_t words = Wb >> 2;
                parts = dist_parts(T, Wb);
                const int32_t part = T >= words ? tid / words : 0;
                double v = 0.0;
                if (part < parts)
                    for (int32_t q = tid - part * words; q < words; q += T) {
                        const int32_t early = (q & ~3) * 4 - (seg - 16);     // > 0: the row's last vector, first `early` bytes not its own
                        const char *at = tile + q * 4;
                        const auto widen = [&](uint32_t raw, double (&x)[kIn]) {
                            if constexpr (kIn == 1) {
                                x[0] = __uint_as_float(raw);
                            } else {
                                x[0] = __uint_as_float(raw << 16);
                                x[1] = __uint_as_float(raw & 0xffff0000u);
                            }
                        };
                        double x0[kIn], s1[kIn], sq[kIn];
                        widen(*reinterpret_cast<const uint32_t *>(at), x0);
#pragma unroll
                        for (int e = 0; e < kIn; ++e) s1[e] = sq[e] = 0.0;
                        constexpr int kRows = 8;                             // requested before the first is used
                        for (int32_t row0 = part; row0 < p.N; row0 += kRows * parts) {
                            uint32_t raw[kRows];
#pragma unroll
                            for (int u = 0; u < kRows; ++u) {
                                const int32_t row = row0 + u * parts;
                                raw[u] = *reinterpret_cast<const uint32_t *>(at + (row < p.N ? row : 0) * Wb);       // (row 0 adds zeros)
                            }
#pragma unroll
                            for (int u = 0; u < kRows; ++u) {
                                double x[kIn];
                                widen(raw[u], x);
#pragma unroll
                                for (int e = 0; e < kIn; ++e) {
                                    const double dlt = x[e] - x0[e];
                                    s1[e] += dlt;
                                    sq[e] = fma(dlt, dlt, sq[e]);
                                }
                            }
                        }
#pragma unroll
                        for (int e = 0; e < kIn; ++e) {
                            if ((q & ~3) * 4 >= seg || (q & 3) * 4 + e * kEs < early) s1[e] = sq[e] = 0.0;
                            if (parts > 1) red[part * columns + q * kIn + e] = s1[e];
                        }
                        const double s2 = kIn == 1 ? sq[0] : sq[0] + sq[kIn - 1];
                        const double t2 = kIn == 1 ? s1[0] * s1[0] : fma(s1[0], s1[0], s1[kIn - 1] * s1[kIn - 1]);
                        v += parts == 1 ? s2 - over(t2, p.peers, p.inv_n) : s2;
                    }
                v = wave_sum(v);
                if (lane == 0) squares[wave] = v;
                if (parts == 1) columns = 0;
            } else {
                const int32_t c = tid & wv_mask, sharers = T >> wv_shift;
                const int32_t early = c * 16 - (seg - 16);
                const int32_t dup = early > 0 ? early / kEs : 0;
                constexpr int kChains = PHASES == 1 ? NE : 1;
                double s1[NE], sq[kChains], s2 = 0.0;
                float x0[NE];
                widen16<DT>(*lds_vec(0, c), x0);
#pragma unroll
                for (int e = 0; e < NE; ++e) s1[e] = 0.0;
#pragma unroll
                for (int e = 0; e < kChains; ++e) sq[e] = 0.0;
                if (c * 16 < seg) {
                    // (four rows are requested before the first is used: LDS latency is what a lone read waits for)
                    constexpr int kRows = PHASES == 1 ? 4 : 1;       // (few registers are free next to 16 slots)
                    for (int32_t row0 = tid >> wv_shift; row0 < p.N; row0 += kRows * sharers) {
                        u32x4 raw[kRows];
#pragma unroll
                        for (int u = 0; u < kRows; ++u) {
                            const int32_t row = row0 + u * sharers;
                            raw[u] = *lds_vec(row < p.N ? row : 0, c);       // (row 0 adds zeros)
                        }
#pragma unroll
                        for (int u = 0; u < kRows; ++u) {
                            float x[NE];
                            widen16<DT>(raw[u], x);
#pragma unroll
                            for (int e = 0; e < NE; ++e) {
                                double dlt = static_cast<double>(x[e]) - static_cast<double>(x0[e]);
                                if (PHASES > 1 && e < dup) dlt = 0.0;
                                s1[e] += dlt;
                                sq[e % kChains] = fma(dlt, dlt, sq[e % kChains]);
                            }
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < kChains; ++e) {
                    if (PHASES == 1 && e < dup) { s1[e] = 0.0; sq[e] = 0.0; }
                    s2 += sq[e];
                }
                column_sums<NE>(s1, s2, wv_shift, red + wave * columns, squares + wave);
            }
            lds_barrier();
            if (wave == entry % waves) {
                const double sum = finish_columns(red, parts, columns, squares, waves, p.peers, p.inv_n);
                if (lane == 0) p.partials[out_at] = sum;
            }
        }
    };

    // Moshpit SGD: rows present in the first round enter as theta - gamma * g
    if (p.grad != nullptr) {
        const char *origin = p.grad + cur.col0;
        int32_t t_ = tid;
        asm volatile("" : "+v"(t_));
        constexpr int kBatch = PHASES == 1 ? kSlots : 4;     // (few registers are free next to 16 slots)
#pragma unroll
        for (int b0 = 0; b0 < kSlots; b0 += kBatch) {
            u32x4 g[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
                g[b] = load_vec<NT, u32x4>(origin + slot_offset(cur, t_ + (b0 + b) * T, p.grad_row_bytes));
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int32_t idx = t_ + (b0 + b) * T;
                if (slot_valid(cur, idx) && (flags[idx >> full_shift] & 2)) {
                    pre[b0 + b] = local_step<DT>(pre[b0 + b], g[b], p.gamma);
                    if constexpr (DT == 0)
#pragma unroll
                        for (int e = 0; e < 4; ++e) pre[b0 + b][e] = __float_as_uint(__uint_as_float(pre[b0 + b][e]) + p.step_zero);
                }
            }
        }
    }

#pragma unroll 1
    for (int32_t phase = 0; phase < PHASES; ++phase) {
        // bytes of this part; with two parts half the lanes hold one, half the other (T is a multiple of a row's vectors)
        const int32_t left = cur.seg - phase * Wb;
        const int32_t seg = left < Wb ? left : Wb;
        const int64_t tiles = p.tiles * PHASES;
        if (seg <= 0) {
            if constexpr (DIST)
                for (int32_t e = tid; e <= p.rounds; e += T)
                    if (e > 0 || p.dist_before) p.partials[e * tiles + w * PHASES + phase] = 0.0;
            break;
        }
        const bool mine = PHASES == 1 || ((tid & full_mask) >> wv_shift) == phase;
        int32_t t_ = tid;
        asm volatile("" : "+v"(t_));
#pragma unroll
        for (int b = 0; b < kSlots; ++b) {
            const int32_t idx = t_ + b * T;
            if (mine && slot_valid(cur, idx)) *lds_vec(idx >> full_shift, idx & wv_mask) = pre[b];
        }
        lds_barrier();

        if constexpr (DIST)
            if (p.dist_before) distortion(seg, 0, w * PHASES + phase);
        int32_t axis = p.axis0;
        for (int32_t r = 0; r < p.rounds; ++r) {
            if (p.copies != nullptr && (r > 0 || p.refresh_first)) {
                // returning peers copy their donors (who do not return themselves)
                const uint32_t *list = p.copies + static_cast<int64_t>(r) * p.N;
                const int32_t items = p.copy_counts[r] << wv_shift;
                for (int32_t it = tid; it < items; it += T) {
                    const uint32_t pair = list[it >> wv_shift];
                    const int32_t v = it & wv_mask;
                    *lds_vec(static_cast<int32_t>(pair & 0xffffu), v) = *lds_vec(static_cast<int32_t>(pair >> 16), v);
                }
                lds_barrier();
            }
            round(seg, axis, bitmaps + r * p.groups);
            lds_barrier();
            if constexpr (DIST)
                if ((p.dist_after >> r) & 1u) distortion(seg, r + 1, (r + 1) * tiles + w * PHASES + phase);
            axis = axis + 1 == p.d ? 0 : axis + 1;
        }
        if constexpr (PHASES == 2) {
            // back into the registers; the next part enters LDS when everybody is done with this one
            t_ = tid;
            asm volatile("" : "+v"(t_));
#pragma unroll
            for (int b = 0; b < kSlots; ++b) {
                const int32_t idx = t_ + b * T;
                if (mine && slot_valid(cur, idx)) pre[b] = *lds_vec(idx >> full_shift, idx & wv_mask);
            }
            if (phase == 0) lds_barrier();
        }
    }

    if (p.rounds > 0) {
        char *origin = X + cur.col0;
        int32_t t_ = tid;
        asm volatile("" : "+v"(t_));
        constexpr int kBatch = 4;
#pragma unroll
        for (int b0 = 0; b0 < kSlots; b0 += kBatch) {
            uint8_t used[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                int32_t idx = t_ + (b0 + b) * T;
                if (!slot_valid(cur, idx)) idx = 0;
                if constexpr (PHASES == 1) pre[b0 + b] = *lds_vec(idx >> full_shift, idx & full_mask);
                used[b] = flags[idx >> full_shift];
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int32_t idx = t_ + (b0 + b) * T;
                if (used[b] != 0 && slot_valid(cur, idx)) store_vec<NT, u32x4>(origin + slot_offset(cur, idx, p.row_bytes), pre[b0 + b]);
            }
        }
    }
}

// out[e] = (sum of partials[e][0 .. tiles)) / n, entry e = blockIdx.x, in a fixed order, for the entries
// that the pass computed
__global__ __launch_bounds__(kSumThreads) void grid_dist_kernel(const double *__restrict__ partials, int64_t tiles, double n,
                                                                int32_t before, uint64_t after, double *__restrict__ out)
{
    if (blockIdx.x == 0 ? before == 0 : ((after >> (blockIdx.x - 1)) & 1u) == 0) return;
    const double sum = block_sum(partials + blockIdx.x * tiles, tiles);
    if (threadIdx.x == 0) out[blockIdx.x] = sum / n;
}

// ---- what a pass needs to know about the peers: one launch per run ----------------------------

// Stable compaction step of one block: number of set flags of the threads before this one; *total the block's.
__device__ __forceinline__ int32_t block_rank(bool flag, int32_t *wave_sums, int32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long ballot = __ballot(flag);
    if (lane == 0) wave_sums[wave] = __popcll(ballot);
    __syncthreads();
    int32_t base = 0, all = 0;
    for (int k = 0; k < kPlanThreads / 64; ++k) {
        const int32_t c = wave_sums[k];
        if (k < wave) base += c;
        all += c;
    }
    __syncthreads();
    *total = all;
    return base + __popcll(ballot & ((1ull << lane) - 1ull));
}

// Blocks 0 .. rounds-1: round r = blockIdx.x: bitmaps[r][g] (bit j: position j of group g takes
// part) and, with refresh, the (donor << 16 | returning peer) pairs of the round.  Blocks after
// that: flags[i] for 1024 peers each (bit 0: takes part in some round or is refreshed; bit 1: in
// the first one).  A die-and-rejoin schedule comes as masks: its walk over the rounds spreads over
// the chip in the schedule kernel, while one block a round that walks for 4096 peers takes 42 us.
__global__ __launch_bounds__(kPlanThreads) void grid_plan_kernel(GridSchedule s, GridTables o)
{
    __shared__ uint8_t here[kGridMaxPeers];
    __shared__ uint16_t candidates[kGridMaxPeers];
    __shared__ int32_t wave_sums[kPlanThreads / 64];
    const int32_t N = s.N, tid = threadIdx.x;
    if (static_cast<int32_t>(blockIdx.x) < s.rounds) {
        const int32_t r = blockIdx.x;
        const int64_t t = s.t0 + r;
        const bool refresh = s.refresh && (r > 0 || s.continued);
        bool was[kPerThread], is[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int32_t i = tid + k * kPlanThreads;
            was[k] = is[k] = false;
            if (i < N) {
                presence(s, i, r, was[k], is[k]);
                here[i] = is[k] ? 1 : 0;
            }
        }
        __syncthreads();
        int64_t S = 1;
        for (int64_t q = 0; q < t % s.d; ++q) S *= s.M;
        const int32_t groups = N / s.M;
        for (int32_t g = tid; g < groups; g += kPlanThreads) {
            const int32_t base = static_cast<int32_t>((g / S) * S * s.M + g % S);
            uint32_t bits = 0;
            for (int32_t j = 0; j < s.M; ++j) bits |= static_cast<uint32_t>(here[base + j * S]) << j;
            if (s.group_skip && static_cast<int32_t>(__popc(bits)) != s.M) bits = 0;
            o.bitmaps[static_cast<int64_t>(r) * groups + g] = bits;
        }
        if (!refresh) {
            if (s.refresh && tid == 0) o.copy_counts[r] = 0;
            return;
        }
        int32_t c = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            int32_t total = 0;
            const bool cand = was[k] && is[k];
            const int32_t rank = block_rank(cand, wave_sums, &total);
            if (cand) candidates[c + rank] = static_cast<uint16_t>(tid + k * kPlanThreads);
            c += total;
        }
        __syncthreads();
        const uint64_t round_key = mix64(s.seed + 0xA0761D6478BD642Full * static_cast<uint64_t>(t + 1));
        int32_t n = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            int32_t total = 0;
            const int32_t i = tid + k * kPlanThreads;
            const bool returns = c > 0 && is[k] && !was[k];
            const int32_t rank = block_rank(returns, wave_sums, &total);
            if (returns) {
                const uint64_t u = mix64(round_key ^ static_cast<uint64_t>(i));
                const uint32_t donor = candidates[u % static_cast<uint64_t>(c)];
                o.copies[static_cast<int64_t>(r) * N + n + rank] = donor << 16 | static_cast<uint32_t>(i);
            }
            n += total;
        }
        if (tid == 0) o.copy_counts[r] = n;
    } else {
        const int32_t i = (static_cast<int32_t>(blockIdx.x) - s.rounds) * kPlanThreads + tid;
        if (i >= N) return;
        uint8_t flag = 0;
        for (int32_t r = 0; r < s.rounds; ++r) {
            const bool now = s.masks != nullptr ? s.masks[static_cast<int64_t>(r) * N + i] != 0
                                                : !failure_event(s.seed, s.t0 + r, i, s.threshold);
            if (now) flag |= r == 0 ? 3 : 1;
        }
        o.flags[i] = flag;
    }
}

// Group-skip schedules without refresh: a peer whose groups all sit out is not touched.
__global__ __launch_bounds__(256) void grid_skip_flags_kernel(GridSchedule s, GridTables o)
{
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= s.N) return;
    const int32_t groups = s.N / s.M;
    uint8_t flag = 0;
    for (int32_t r = 0; r < s.rounds; ++r) {
        int32_t S = 1;
        for (int64_t q = 0; q < (s.t0 + r) % s.d; ++q) S *= s.M;
        const int32_t g = i / (S * s.M) * S + i % S, j = i / S % s.M;
        if ((o.bitmaps[static_cast<int64_t>(r) * groups + g] >> j) & 1u) flag |= r == 0 ? 3 : 1;
    }
    if (s.refresh) flag |= o.flags[i] & 1;           // a refreshed peer is written although its group sits out
    o.flags[i] = flag;
}

}  // namespace

hipError_t launch_grid_plan(const GridSchedule &s, const GridTables &tables, hipStream_t stream)
{
    if (s.rounds <= 0) return hipSuccess;
    const uint32_t blocks = static_cast<uint32_t>(s.rounds + (s.N + kPlanThreads - 1) / kPlanThreads);
    grid_plan_kernel<<<dim3(blocks), dim3(kPlanThreads), 0, stream>>>(s, tables);
    if (s.group_skip)
        grid_skip_flags_kernel<<<dim3((s.N + 255) / 256), dim3(256), 0, stream>>>(s, tables);
    return hipGetLastError();
}

namespace {

typedef void (*grid_kernel_t)(char *, GridPlan);

template <int DT, int TREE, int SPLIT, int PER> grid_kernel_t pick_mode(bool two, bool nt, bool dist)
{
    if (two) return nt ? (dist ? grid_rounds_kernel<DT, TREE, SPLIT, PER, 2, true, true> : grid_rounds_kernel<DT, TREE, SPLIT, PER, 2, true, false>)
                       : (dist ? grid_rounds_kernel<DT, TREE, SPLIT, PER, 2, false, true> : grid_rounds_kernel<DT, TREE, SPLIT, PER, 2, false, false>);
    return nt ? (dist ? grid_rounds_kernel<DT, TREE, SPLIT, PER, 1, true, true> : grid_rounds_kernel<DT, TREE, SPLIT, PER, 1, true, false>)
              : (dist ? grid_rounds_kernel<DT, TREE, SPLIT, PER, 1, false, true> : grid_rounds_kernel<DT, TREE, SPLIT, PER, 1, false, false>);
}

grid_kernel_t pick_kernel(int dtype, const GridPlan &p, bool dist)
{
    const bool two = p.phases == 2, nt = p.streaming != 0;
    if (dtype == 0) {
        if (p.M <= 2) return pick_mode<0, 2, 1, 0>(two, nt, dist);
        if (p.M <= 4) return pick_mode<0, 4, 1, 0>(two, nt, dist);
        if (p.M <= 8) return pick_mode<0, 8, 1, 0>(two, nt, dist);
        if (p.M <= 16) return pick_mode<0, 16, 2, 8>(two, nt, dist);
        return pick_mode<0, 16, 4, 8>(two, nt, dist);
    }
    if (p.M <= 2) return pick_mode<1, 2, 1, 0>(two, nt, dist);
    if (p.M <= 4) return pick_mode<1, 4, 1, 0>(two, nt, dist);
    if (p.M <= 8) return pick_mode<1, 8, 1, 0>(two, nt, dist);
    if (p.M <= 16) return pick_mode<1, 16, 1, 0>(two, nt, dist);
    return pick_mode<1, 16, 4, 8>(two, nt, dist);
}

}  // namespace

hipError_t launch_grid_rounds(void *X, int dtype, const GridPlan &plan, hipStream_t stream)
{
    GridPlan p = plan;
    const bool dist = p.partials != nullptr;
    p.lds_bytes = static_cast<int32_t>(copies_lds_bytes(p, p.rounds, dist, dtype == 0 ? 4 : 2, &p.red_offset));
    if (p.lds_bytes > kLdsPerBlock || p.tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const grid_kernel_t kernel = pick_kernel(dtype, p, dist);
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), kLdsPerBlock);
    if (e != hipSuccess) return e;
    kernel<<<dim3(static_cast<uint32_t>(p.tiles)), dim3(p.threads), p.lds_bytes, stream>>>(static_cast<char *>(X), p);
    return hipGetLastError();
}

hipError_t launch_grid_dist(const GridPlan &p, double *out, hipStream_t stream)
{
    const int64_t tiles = p.tiles * p.phases;
    grid_dist_kernel<<<dim3(static_cast<uint32_t>(p.rounds + 1)), dim3(sum_threads(tiles)), 0, stream>>>(
        p.partials, tiles, static_cast<double>(p.N), p.dist_before, p.dist_after, out);
    return hipGetLastError();
}

}  // namespace moshpit
