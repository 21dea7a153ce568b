// Group-mean round kernel for gfx950 (MI355X).
//
// One averaging round of Moshpit All-Reduce (Alg. 1, the AllReduce line; the
// group-average formula of App. C.3 with the group J_{i,t} of App. C.4) on N
// virtual peers stored as rows of X.  For round t the group g owns the M rows
// base(g) + j*S, S = M^(t mod d); every row whose peer takes part is replaced
// by the mean of the rows that take part.
//
// Mapping.  The reduction runs ACROSS rows, so each lane owns its columns for
// the whole group and no cross-lane traffic or LDS is needed: a work item is
// (group, column tile); a thread loads one 128-bit vector per participating
// row (COLS of them, 256 lanes apart, to keep more loads in flight when M is
// small), sums in binary32 registers, divides by the participant count and
// stores the mean to the same rows.  Rows of absent peers are never touched,
// so HBM traffic is 2 * elem_size * P bytes per participating peer.  In-place
// is safe because a work item reads and writes only its own (group, tile) and
// all its loads retire before its first store.
//
// The participant bitmap of a group is built by the wave itself: lane j < M
// reads alive[base + j*S] and a ballot gives a 64-bit mask (hence M <= 64).  A
// host mask of up to 4096 peers arrives as kernel arguments instead, its bits in
// group order, and costs the wave two scalar loads: no copy to the device and no
// event per round (27 peers x 1,001 bfloat16: 12.7 -> 5.4 us a round; 8 x 8 x 8 x
// 8,869: 17.9 -> 7.8).
#include "moshpit_internal.h"
#include "row_vec.h"

namespace moshpit {
namespace {

constexpr int kMaxBlock = 256;          // threads per block: 64, 128 or 256
constexpr int kLdsPerCu = 160 * 1024;   // gfx950: LDS bytes per compute unit

// X            state, byte pointer to element (row 0, first column of this launch)
// row_bytes    distance between rows in bytes
// valid_bytes  bytes of a row; nvec = ceil(valid_bytes / vector size) vectors of VE elements.
//              Rows may start on any element.  Where a row is not a whole number of vectors its
//              last vector ends with the row and shares columns with its neighbour; both are
//              averaged, with the same bits.  The two always belong to one work item of one wave
//              (a work item that would start with that last vector starts one vector earlier),
//              whose loads all come before its stores.
// tiles        ceil(nvec / (blockDim.x * COLS))
// work_items   groups * tiles
// bits         BITS: who takes part as kernel arguments (instead of alive), group by group: bit j of
//              group g at position g * M + j
// IDX          groups are consecutive chunks of M entries of the peer list
//              index[0..n_index) (e.g. a random permutation) instead of grid lines
// SGD          the Moshpit SGD communication step (Alg. 2): what is averaged is
//              theta_j - gamma * g_j, g read from the matrix G laid out like X
//              (rows g_row_bytes apart); a peer that is alone in its group still
//              takes its local step
struct NoBits {};
// BITS: 0 none, 1 up to kFewPeers peers, 2 up to kSmallOrderPeers
template <int BITS> struct BitsOf;
template <> struct BitsOf<0> { typedef NoBits type; };
template <> struct BitsOf<1> { typedef FewPeerBits type; };
template <> struct BitsOf<2> { typedef PeerBits type; };

template <int DT, int VE, int COLS, int U, bool NT, bool IDX, bool SGD, int BITS>
__global__ __launch_bounds__(kMaxBlock) void group_mean_kernel(char *X, int64_t row_bytes, int64_t valid_bytes,
                                                            const uint8_t *__restrict__ alive, int32_t M,
                                                            int64_t S, int64_t tiles, int64_t work_items,
                                                            const int32_t *__restrict__ index, int64_t n_index,
                                                            const int32_t *__restrict__ n_groups,
                                                            const char *__restrict__ G, int64_t g_row_bytes,
                                                            float gamma, int order,
                                                            typename BitsOf<BITS>::type bits)
{
    typedef Vec<DT, VE> V;
    typedef typename V::mem_t mem_t;
    constexpr int NE = V::NE;
    const int lane = threadIdx.x & 63;
    const int kBlock = blockDim.x;
    constexpr int64_t kVec = sizeof(mem_t);
    // order 1: blocks b, b + 8, b + 16, ... (they run on the same one of the 8 dies) take
    // consecutive work items: each die streams through an eighth of the list.  The eighths are
    // rounded up, so there are 8 * per places, a block for each, and the last ones may hold no item.
    int64_t w0 = blockIdx.x;
    do {
        int64_t w = w0;
        if (order == 1) {
            const int64_t per = (work_items + 7) >> 3;
            w = (w0 & 7) * per + (w0 >> 3);
            if (w >= work_items) break;
        } else if (order > 1) {
            // runs of 2^order: a die takes so many of every eight times as many, and an eighth of what is left at the end
            const int64_t span = int64_t(8) << order, first = w0 & ~(span - 1), r = w0 - first, left = work_items - first;
            const int64_t run = (left < span ? left : span) >> 3;
            if (r < 8 * run) w = first + (r & 7) * run + (r >> 3);
        }
        const int64_t g = w / tiles;
        const int64_t tile = w - g * tiles;
        int64_t base = 0;
        int32_t my_row = -1;                         // IDX: the row of position `lane`
        bool takes_part = false;
        if constexpr (IDX) {
            const int64_t pos = g * M + lane;
            if (lane < M && pos < n_index) my_row = index[pos];
            takes_part = my_row >= 0 && ((alive == nullptr) || (alive[my_row] != 0));
        } else {
            base = (g / S) * S * M + (g % S);
            if (BITS == 0 && lane < M) takes_part = (alive == nullptr) || (alive[base + static_cast<int64_t>(lane) * S] != 0);
        }
        uint64_t live = __ballot(takes_part);
        if constexpr (BITS != 0) {
            // (g is uniform: two or three words of the argument block through the scalar cache)
            const uint32_t first = static_cast<uint32_t>(g) * static_cast<uint32_t>(M), at = first >> 5, shift = first & 31;
            constexpr uint32_t kWords = sizeof(bits) / 4;
            const auto word = [&](uint32_t k) -> uint64_t { return k < kWords ? bits.word[k] : 0u; };
            live = (word(at) | word(at + 1) << 32) >> shift;
            if (shift != 0 && M > 32) live |= word(at + 2) << (64 - shift);
            if (M < 64) live &= (1ull << M) - 1ull;
        }
        const int cnt = __popcll(live);
        if (cnt < (SGD ? 1 : 2)) continue;           // nothing to do: rows stay as they are

        // (only now: a work item of an empty group ends as soon as its mask is known)
        int64_t bytes = valid_bytes;
        asm volatile("" : "+s"(bytes));
        const int64_t nvec = (bytes + kVec - 1) / kVec;
        int64_t v0 = tile * (static_cast<int64_t>(kBlock) * COLS) + threadIdx.x, v_end = nvec;
        // the ragged last vector would be a work item of its own
        if (bytes % kVec != 0 && tiles > 1 && nvec == (tiles - 1) * kBlock * COLS + 1) {
            if (tile == tiles - 1) v0 -= 1;
            else if (tile == tiles - 2) v_end -= 2;
        }
        bool in_row[COLS];
        int64_t at[COLS];                            // byte of the row where this lane's vector starts
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            const int64_t v = v0 + c * kBlock;
            in_row[c] = v < v_end;
            at[c] = v * kVec < valid_bytes - kVec ? v * kVec : valid_bytes - kVec;
        }

        char *gbase = X + base * row_bytes;
        const int64_t jstep = S * row_bytes;
        // first byte of the row of position j (j is wave-uniform)
        auto row_ptr = [&](int j) -> char * {
            if constexpr (IDX)
                return gbase + static_cast<int64_t>(__builtin_amdgcn_readlane(my_row, j)) * row_bytes;
            else
                return gbase + j * jstep;
        };

        float acc[COLS][NE];
#pragma unroll
        for (int c = 0; c < COLS; ++c)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[c][e] = 0.f;

        // Rows are taken in chunks of U by POSITION j (absent rows contribute an
        // exact 0 and cost no load), so the summation order is a fixed balanced
        // tree over the M slots whatever the mask: ((x0+x1)+(x2+x3))+... per
        // chunk, chunks added in ascending order.
        for (int j0 = 0; j0 < M; j0 += U) {
            const uint64_t bits = (live >> j0) & (U >= 64 ? ~0ull : ((1ull << (U % 64)) - 1ull));
            if (bits == 0) continue;
            mem_t buf[U][COLS];
            mem_t gbuf[SGD ? U : 1][COLS];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int c = 0; c < COLS; ++c) {
                    buf[u][c] = V::zero();
                    if constexpr (SGD) gbuf[u][c] = V::zero();
                }
                if ((bits >> u) & 1ull) {
                    const char *src = row_ptr(j0 + u);
#pragma unroll
                    for (int c = 0; c < COLS; ++c)
                        if (in_row[c]) buf[u][c] = load_vec<NT, mem_t>(src + at[c]);
                    if constexpr (SGD) {
                        const char *gsrc = G + (base + (j0 + u) * S) * g_row_bytes;
#pragma unroll
                        for (int c = 0; c < COLS; ++c)
                            if (in_row[c]) gbuf[u][c] = load_vec<NT, mem_t>(gsrc + at[c]);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < COLS; ++c) {
                float f[U][NE];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    V::widen(buf[u][c], f[u]);
                    if constexpr (SGD) {
                        float gf[NE];
                        V::widen(gbuf[u][c], gf);
#pragma unroll
                        for (int e = 0; e < NE; ++e) f[u][e] = fmaf(-gamma, gf[e], f[u][e]);
                    }
                }
#pragma unroll
                for (int s = 1; s < U; s *= 2)
#pragma unroll
                    for (int u = 0; u + s < U; u += 2 * s)
#pragma unroll
                        for (int e = 0; e < NE; ++e) f[u][e] += f[u + s][e];
#pragma unroll
                for (int e = 0; e < NE; ++e) acc[c][e] += f[0][e];
            }
        }

        const float k = static_cast<float>(cnt);
        mem_t mean[COLS];
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[c][e] = acc[c][e] / k;
            mean[c] = V::narrow(acc[c]);
        }

        uint64_t rem = live;
        while (rem != 0) {
            const int j = __builtin_ctzll(rem);
            rem &= rem - 1;
            char *dst = row_ptr(j);
#pragma unroll
            for (int c = 0; c < COLS; ++c)
                if (in_row[c]) store_vec<NT, mem_t>(dst + at[c], mean[c]);
        }
        // (a run's places up to its end: they are in another order than its work items)
    } while ((w0 += gridDim.x) < work_items &&
             (!IDX || n_groups == nullptr || (order > 1 ? w0 >> (order + 3) << (order + 3) : w0) < *n_groups * tiles));
}

// The kernel uses no LDS.  The dynamic-LDS size of the launch is only a
// throttle: a block that reserves lds bytes lets floor(160 KiB / lds) blocks
// share a compute unit, which bounds the number of row loads in flight.
template <int DT, int VE, int COLS, int U, bool NT, bool IDX = false, bool SGD = false, int BITS = 0>
hipError_t launch_one(char *X, int64_t row_bytes, int64_t valid_bytes, const uint8_t *alive, const RoundGeom &geom,
                      int block, int waves_per_cu, int order, hipStream_t stream)
{
    constexpr int64_t kVec = VE * (DT == 0 ? 4 : 2);
    if (valid_bytes < kVec) return hipErrorInvalidValue;
    const int64_t nvec = (valid_bytes + kVec - 1) / kVec;
    if (valid_bytes % kVec != 0) block = 64;         // the last two vectors of a row belong to one wave
    const int64_t per_tile = static_cast<int64_t>(block) * COLS;
    const int64_t tiles = (nvec + per_tile - 1) / per_tile;
    const int64_t groups = IDX ? (geom.n_index + geom.M - 1) / geom.M : geom.N / geom.M;
    const int64_t work = groups * tiles;
    if (work <= 0) return hipSuccess;
    int64_t grid = work < 0x7fffffffLL ? work : 0x7fffffffLL;
    // A list with room for part-filled groups, as chunk-index rounds give, is half empty.  Where its work items come in many
    // turns, blocks for those that fill it when everybody takes part do; a block goes on to another if there is one
    // (16 x 16 x 16 x 6,824 binary32 56 us a round with a block for every place, 45 so; but 8 x 8 x 8 x 3,712 bfloat16, 512
    // work items, 11.7 and 12.5).
    const int64_t full = geom.N / geom.M * tiles;
    if (IDX && geom.n_groups != nullptr && full >= 8192 && full < grid) grid = full;
    if (order == 1) {
        grid = ((work + 7) >> 3) << 3;
        if (grid > 0x7fffffffLL) { grid = 0x7fffffffLL; order = 0; }    // (more work items than blocks: plain order)
    }
    auto kernel = group_mean_kernel<DT, VE, COLS, U, NT, IDX, SGD, BITS>;
    typename BitsOf<BITS>::type bits{};
    if constexpr (BITS == 1) bits = few_bits(*geom.bits);
    else if constexpr (BITS == 2) bits = *geom.bits;
    size_t lds = 0;
    if (waves_per_cu > 0 && waves_per_cu < 32) {
        int blocks_per_cu = waves_per_cu / (block / 64);
        if (blocks_per_cu < 1) blocks_per_cu = 1;
        lds = lds_bytes_for_blocks_per_cu(blocks_per_cu);
        hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), kLdsPerCu);
        if (e != hipSuccess) return e;
    }
    kernel<<<dim3(static_cast<uint32_t>(grid)), dim3(block), lds, stream>>>(X, row_bytes, valid_bytes, alive, geom.M,
                                                                            geom.S, tiles, work, geom.index,
                                                                            geom.n_index, geom.n_groups, geom.grad, geom.grad_row_bytes,
                                                                            geom.gamma, order, bits);
    return hipGetLastError();
}

template <int DT, int VE>
hipError_t launch_shape(int cols, int unroll, bool nt, char *X, int64_t row_bytes, int64_t valid_bytes,
                        const uint8_t *alive, const RoundGeom &geom, int block, int wpc, int order, hipStream_t stream)
{
    if (geom.bits != nullptr) {
        // a host mask of up to 4096 peers: the default shapes only
        const bool few = geom.N <= kFewPeers;
#define MOSHPIT_BITS_OF(C, UU, B)                                                                                       \
            return nt ? launch_one<DT, VE, C, UU, true, false, false, B>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream) \
                      : launch_one<DT, VE, C, UU, false, false, false, B>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
#define MOSHPIT_BITS(C, UU)                                                                                             \
        if (cols == C && unroll == UU) {                                                                               \
            if (few) MOSHPIT_BITS_OF(C, UU, 1)                                                                          \
            MOSHPIT_BITS_OF(C, UU, 2)                                                                                   \
        }
        MOSHPIT_BITS(1, 16)
        MOSHPIT_BITS(2, 8)
        MOSHPIT_BITS(1, 4)
        MOSHPIT_BITS(4, 2)
#undef MOSHPIT_BITS
#undef MOSHPIT_BITS_OF
        return hipErrorInvalidValue;
    }
    if (geom.index != nullptr) {
        // peer-list groups: the default shapes only
        if (cols == 1 && unroll == 16) return nt ? launch_one<DT, VE, 1, 16, true, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 1, 16, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 2 && unroll == 8) return nt ? launch_one<DT, VE, 2, 8, true, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 2, 8, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 4 && unroll == 4) return nt ? launch_one<DT, VE, 4, 4, true, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 4, 4, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 4 && unroll == 2) return nt ? launch_one<DT, VE, 4, 2, true, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 4, 2, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        return hipErrorInvalidValue;
    }
    if (geom.grad != nullptr) {
        // Moshpit SGD step: the default shapes only
        if (cols == 1 && unroll == 16) return nt ? launch_one<DT, VE, 1, 16, true, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 1, 16, false, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 2 && unroll == 8) return nt ? launch_one<DT, VE, 2, 8, true, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 2, 8, false, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 4 && unroll == 4) return nt ? launch_one<DT, VE, 4, 4, true, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 4, 4, false, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        if (cols == 4 && unroll == 2) return nt ? launch_one<DT, VE, 4, 2, true, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                                                  : launch_one<DT, VE, 4, 2, false, false, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
        return hipErrorInvalidValue;
    }
#define MOSHPIT_CASE(C, UU)                                                                          \
    if (cols == C && unroll == UU)                                                                   \
        return nt ? launch_one<DT, VE, C, UU, true>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)   \
                  : launch_one<DT, VE, C, UU, false>(X, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
    MOSHPIT_CASE(1, 4)
    MOSHPIT_CASE(1, 8)
    MOSHPIT_CASE(1, 16)
    MOSHPIT_CASE(1, 32)
    MOSHPIT_CASE(2, 2)
    MOSHPIT_CASE(2, 4)
    MOSHPIT_CASE(2, 8)
    MOSHPIT_CASE(2, 16)
    MOSHPIT_CASE(4, 2)
    MOSHPIT_CASE(4, 4)
    MOSHPIT_CASE(4, 8)
#undef MOSHPIT_CASE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_group_mean(void *X, int dtype, int64_t P, int64_t row_stride, const RoundGeom &geom,
                             const uint8_t *alive, const MeanTuning &tune, hipStream_t stream)
{
    const int64_t esize = dtype == 0 ? 4 : 2;
    const int64_t row_bytes = row_stride * esize;
    const int64_t valid_bytes = P * esize;

    // Defaults (measured on MI355X over block sizes, rows in flight and resident waves):
    // one-wave blocks, each wave keeps about 16 KiB of row loads in flight
    // (rows per chunk x cols x 1 KiB) and 4-7 waves share a compute unit, i.e.
    // about 16-28 MiB in flight on the chip.  More than that and the HBM
    // controllers see too many open pages; less and latency is not covered.
    int cols = tune.cols, unroll = tune.unroll;
    if (cols <= 0 || unroll <= 0 || geom.bits != nullptr || geom.index != nullptr || geom.grad != nullptr) {
        if (geom.M > 8) { unroll = 16; cols = 1; }
        else if (geom.M > 4) { unroll = 8; cols = 2; }
        else if (geom.M > 2) {
            // four rows per group: one vector per row and lane and 20 resident waves measured 2 %
            // above four vectors and 5 waves on 100 MB rows (peer lists and the SGD step keep four)
            unroll = 4;
            cols = (geom.index != nullptr || geom.grad != nullptr) ? 4 : 1;
        }
        else { unroll = 2; cols = 4; }
    }
    // Non-temporal or ordinary accesses (measured on MI355X; GB/s are bytes of one round over its time).
    // Non-temporal ones are worth 3 - 17 % where a large state streams through (1 GiB, 16 x 16
    // peers: 5.6 against 5.3 TB/s).  A state of up to 256 MiB stays in the last-level cache from
    // round to round if the accesses are ordinary, and wants more waves in flight, since its latency
    // is what limits: 256 MiB, 16 x 16 peers 5.4 -> 6.2 TB/s, 64 MiB 4.1 -> 4.7, 32 x 32 peers of
    // 128 MiB 4.5 -> 5.7, 4 x 4 x 4 of 256 MiB 5.4 -> 6.4; at 512 MiB both are equal, and below
    // the L2s' 32 MiB the non-temporal ones are ahead by 5 %.  Rows that
    // do not start on cache lines share their first and last lines with other work items: the parts
    // have to meet in L2 (16 x 16 peers x 2,000,001 binary32: 4.5 -> 5.3 TB/s, x 1,200,007
    // bfloat16: 4.3 -> 5.2, 4 x 4 x 4 x 9,000,001: 4.7 -> 5.6).
    const double touched = static_cast<double>(geom.N) * row_bytes * (geom.grad != nullptr ? 2 : 1);
    const bool whole_lines = reinterpret_cast<uintptr_t>(X) % 128 == 0 && row_bytes % 128 == 0;
    // (off the cache lines that holds longer: 12 x 12 peers x 630,769 binary32, 347 MiB, 5.7 -> 6.1 TB/s;
    // at 381 MiB, everybody present, groups of 7 to 32 rows are within 3 % of what larger states take, 5 rows
    // would gain 9 % from their rules)
    const bool cached = touched <= (whole_lines ? 256.0 : 448.0) * (1 << 20);
    // Peer lists, whose rows lie apart and come back in other groups, hold on to it longer, with ordinary accesses and more waves.  Time of
    // non-temporal accesses over that, chunk-index and random rounds with 10 % absent, both types: groups of 3 to 8 (8 x 8 x 8, 5 x 5 x 5, 4 x 4 x 4,
    // 3^4) at 315 MiB 1.07 to 1.18, 448 1.03 to 1.08, 512 0.99 to 1.03, 534 0.99 to 1.01, 553 0.98 to 1.02, 610 0.96 to 1.01; of 12 to 32 (12 x 12, 16 x 16, 16 x 16 x 16,
    // 32 x 32) at 448 MiB 1.04 to 1.12, 512 0.99 to 1.09, 553 1.01 to 1.07, 572 1.01 to 1.07, 610 0.98 to 1.05, 686 0.96 to 1.04.
    const bool cached_list = geom.index != nullptr && whole_lines && !cached && touched <= (geom.M > 8 ? 600.0 : 544.0) * (1 << 20);
    // Rounds over rows off the cache lines, of a state too large for the last-level cache, deal work items to the dies in runs
    // of 32: the first and last lines of a row's part meet in one L2, and the waves in flight still stream a handful of groups.
    const bool runs = !whole_lines && !cached;
    const bool full = (alive == nullptr && geom.bits == nullptr) || geom.present >= 0.97f;
    const bool large_odd = !whole_lines && dtype == 0 && !cached && (geom.M > 16 || touched > 800.0 * (1 << 20));
    // (the SGD step on groups of up to 8 rows streams so few rows at once that non-temporal accesses
    // stay ahead there: 4 x 4 x 4 peers x 15,609,540 binary32 2.15 against 2.47 ms.  So do groups of up to 6 rows in runs,
    // 3^4 of 3 GB binary32 1,042 : 1,123 us, 5 x 5 x 5 bfloat16 1,051 : 1,101, and 8 of large binary32 states, 8 x 8 x 12,000,007 985 : 1,015, but
    // 500 MB 167 : 153)
    const bool lines_meet = !whole_lines && (geom.grad != nullptr ? geom.M > 8
                                             : !(runs && (geom.M <= 6 || (geom.M <= 8 && large_odd && geom.index == nullptr))));
    const bool nt = tune.nt >= 0 ? tune.nt != 0 : (cached ? whole_lines && touched <= 24.0 * (1 << 20) : !lines_meet && !cached_list);
    const int block = (tune.block == 64 || tune.block == 128 || tune.block == 256) ? tune.block : 64;
    // Block order (measured on MI355X over row sizes of 128 KiB .. 32 MiB, groups of 16 and of
    // 32 rows).  Work items go to the blocks tile-fastest, so the waves in flight stream a
    // handful of groups: up to 6.4 TB/s when the byte distance between the rows of a group
    // spreads well over the memory channels, 4.3 - 5.4 TB/s when it is 4, 8 or 16 MiB with 16
    // rows per group (2 MiB with 32).  For those distances each die is given an eighth of the
    // work list to stream through (8 times as many row streams in flight): 5.7 - 5.8 TB/s
    // whatever the distance, below the good cases of the plain order, above its bad ones.
    int order = tune.order;
    if (order < 0) {
        order = 0;
        // A list with room for part-filled groups, as chunk-index rounds give, ends in empty ones: dealt to the
        // dies in eighths it would leave half of them idle (16 x 16 x 390,625 binary32 149 us, 224 in eighths).
        const bool holes = geom.index != nullptr && geom.n_index > geom.N;
        if (runs) {
            // 0.5 to 3 GB with 10 % absent, in whichever of the other two orders was the better : in runs: 8 x 8 x 12,000,007 1,043 : 985 us,
            // 16 x 16 x 2,929,687 1,051 : 1,027, 16 x 16 x 16 x 366,211 bfloat16 1,106 : 1,016, 32 x 32 x 732,422 1,092 : 1,029,
            // 20 x 20 x 312,500, everybody present, 196 : 173; groups of 2 to 40 rows 1.02 to 1.14 times as fast, of 8 binary32 rows
            // with everybody present 1.00.  Peer lists 4 x 4 x 4 x 9,765,625 832 : 806, 16 x 16 x 2,441,406 877 : 858, 32 x 32 x 610,352, part-filled,
            // 967 : 932; SGD steps in groups of 16 x 16 x 16 x 152,588 2,172 : 2,140, 8 x 8 x 19,531,250 bfloat16 2,158 : 2,111.
            order = 5;
        } else if (holes) {
            order = 0;
        } else if (cached) {
            // In eighths from groups of more than 8 rows (16 x 16 x 62,501 binary32, 64 MB: 25.9 us in the plain
            // order, 22.7 in eighths), except for states of up to 24 MiB, whose few work items would leave some
            // dies waiting: 16 MB of 16 x 16 peers 11.3 and 15.2, of 32 x 32 8.3 and 15.4 (on whole cache
            // lines 7.5 and 11.6); 32 MB of 16 x 16 15.4 and 13.9.  With gradients or a peer list that ends sooner;
            // 6 to 10 MiB in groups of up to 16 rows off the cache lines are ahead in eighths (16 x 16 x 7,813 8.8 and 8.4).
            const double state = static_cast<double>(geom.N) * row_bytes / (1 << 20);
            const double plain = geom.grad == nullptr && geom.index == nullptr ? 24.0 : geom.M > 16 ? 18.0 : geom.grad != nullptr ? 14.0 : 6.0;
            const bool ahead = geom.M <= 16 && !whole_lines && state > 6.0 && state <= 10.0;
            order = geom.M > 8 && (state > plain || ahead) ? 1 : 0;
        } else if (geom.index == nullptr) {
            const int64_t member_stride = geom.S * row_bytes;
            const int64_t MiB = 1 << 20;
            // (only where the distance is a multiple of 256 KiB: 16 x 16 peers x 2,000,000 binary32,
            // 8,000,000 bytes apart, runs at 5.95 TB/s in the plain order and 5.56 in this one)
            if (member_stride % (MiB / 4) != 0) order = 0;
            else if (geom.M <= 16 ? (member_stride >= 4 * MiB && member_stride <= 16 * MiB)
                             : (member_stride >= 2 * MiB && member_stride < 4 * MiB))
                order = 1;
        }
    }
    int wpc = tune.waves_per_cu;
    if (wpc <= 0) {
        // Resident waves per compute unit (measured; the optimum is sharp: on 16 MiB rows in
        // groups of 32, 4 waves give 6.1 TB/s, 3 give 5.8 and 5 give 5.9).  A wave keeps
        // rows x cols KiB of loads in flight (twice that with the gradients of the SGD step).
        const int rows = geom.M < unroll ? geom.M : unroll;
        const int kib_per_wave = rows * cols * (block / 64) * (geom.grad != nullptr ? 2 : 1);
        wpc = (dtype == 0 ? 64 : 80) / kib_per_wave * (block / 64);
        // groups of up to 16 rows (16 KiB in flight per wave): 5 waves; 7 when the rows are
        // shorter than 1 MiB and when every die streams its own part of the list; 5 for groups given as a
        // peer list (16 x 16 x 1,048,576 binary32 344 us, 7 waves 354; 16 x 16 x 16 x 65,536 380 and 394) and for
        // the Moshpit SGD step (which also streams the gradients)
        // The figures above and below were measured with 5 - 20 % of the peers absent.  When
        // (nearly) every peer takes part each wave has more loads in flight and fewer waves do
        // better (16 MiB rows in groups of 32: 3 waves 6.2 TB/s, 4 waves 5.8).
        if (wpc < 4) wpc = 4;
        if (full && geom.grad == nullptr && geom.index == nullptr) wpc -= 1;
        if (rows == 16 && cols == 1 && geom.M <= 16) {
            if (geom.grad != nullptr || geom.index != nullptr) wpc = 5;
            else if (full) wpc = order == 1 ? 6 : 5;
            else wpc = (order == 1 || row_bytes < (1 << 20)) ? 7 : 5;
        }
        // groups of up to 4 rows with one vector per row and lane (4 KiB in flight per wave)
        if (rows * cols <= 4) wpc = full ? 14 : 21;
        // ordinary accesses (see above): more in flight, 8 for bfloat16 rows off the cache lines
        if (cached) wpc = geom.M > 8 ? 12 : 16;
        else if (cached_list) wpc = geom.M > 8 ? 8 : 10;
        else if (!whole_lines && geom.grad == nullptr && rows * cols <= 4) wpc = 16;
        // (in runs, a mask as bits: 8 x 8 x 12,000,007 3 waves 985 us, 6 waves 1,022; 16 x 16 x 488,281 3 waves 168, 8 waves 153; 20 x 20 x
        // 625,000 bfloat16 4 waves 175, 8 waves 159; 9 x 9 x 6,172,839 8 waves 706, 11 waves 675, 14 x 14 as fast with either; 32 x 32 x 732,422 3 waves 1,029, 8 waves 1,059; 40 x 40 x 312,455 bfloat16
        // 4 waves 348, 8 waves 360)
        else if (runs && geom.index != nullptr && geom.M > 6 && geom.M <= 24) wpc = 8;
        else if (runs && geom.grad == nullptr && geom.index == nullptr && geom.M > 6)
            wpc = geom.M > 24 ? (dtype == 0 ? 3 : 4) : geom.M <= 8 && large_odd ? 3 : geom.M > 8 && geom.M <= 11 ? 11 : 8;
        else if (!whole_lines && dtype == 1 && geom.M > 8 && geom.M <= 16) wpc = 128 / rows;
        else if (large_odd && geom.grad != nullptr && geom.M > 8 && geom.M <= 16) wpc = 5;
        // (5 x 5 x 5 x 2,000,001 8 waves 343 us, 4 waves 352; a wave whose mask came with its arguments starts loading sooner)
        else if (runs && large_odd && full && geom.M > 4 && geom.grad == nullptr && geom.index == nullptr) wpc = 8;
        else if (runs && dtype == 0 && geom.bits != nullptr && geom.M > 4) wpc = 52 / kib_per_wave;
        if (wpc > 32) wpc = 32;
    }

    char *base = static_cast<char *>(X);
    if (valid_bytes >= 16)
        return dtype == 0 ? launch_shape<0, 4>(cols, unroll, nt, base, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream)
                          : launch_shape<1, 8>(cols, unroll, nt, base, row_bytes, valid_bytes, alive, geom, block, wpc, order, stream);
    // rows of less than one vector, element by element
    if (geom.grad != nullptr)
        return dtype == 0 ? launch_one<0, 1, 1, 16, false, false, true>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream)
                          : launch_one<1, 1, 1, 16, false, false, true>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream);
    if (geom.index != nullptr)
        return dtype == 0 ? launch_one<0, 1, 1, 16, false, true>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream)
                          : launch_one<1, 1, 1, 16, false, true>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream);
    if (geom.bits != nullptr)
        return dtype == 0 ? launch_one<0, 1, 1, 16, false, false, false, 2>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream)
                          : launch_one<1, 1, 1, 16, false, false, false, 2>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream);
    return dtype == 0 ? launch_one<0, 1, 1, 16, false>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream)
                      : launch_one<1, 1, 1, 16, false>(base, row_bytes, valid_bytes, alive, geom, 64, 32, 0, stream);
}

// ---- local iteration of Moshpit SGD (Alg. 2): theta_i <- theta_i - gamma * g_i ----

namespace {
// A lane takes one 16-byte vector of a row, or the elements after the row's last whole vector.
template <int DT, int VE>
__global__ __launch_bounds__(256) void local_step_kernel(char *X, int64_t row_bytes, const char *__restrict__ G,
                                                         int64_t g_row_bytes, int64_t P,
                                                         const uint8_t *__restrict__ alive, float gamma, int64_t tiles)
{
    typedef Vec<DT, VE> V;
    typedef typename V::mem_t mem_t;
    typedef Vec<DT, 1> V1;
    typedef typename V1::mem_t mem1_t;
    constexpr int NE = V::NE;
    const int64_t row = blockIdx.x / tiles;
    const int64_t tile = blockIdx.x - row * tiles;
    if (alive != nullptr && alive[row] == 0) return;
    const int64_t first = (tile * 256 + threadIdx.x) * VE;      // first column of this lane
    if (first >= P) return;
    char *x = X + row * row_bytes + first * static_cast<int64_t>(sizeof(mem1_t));
    const char *g = G + row * g_row_bytes + first * static_cast<int64_t>(sizeof(mem1_t));
    if (first + VE <= P) {
        float xf[NE], gf[NE];
        V::widen(load_vec<true, mem_t>(x), xf);
        V::widen(load_vec<true, mem_t>(g), gf);
#pragma unroll
        for (int e = 0; e < NE; ++e) xf[e] = fmaf(-gamma, gf[e], xf[e]);
        store_vec<true, mem_t>(x, V::narrow(xf));
    } else {
        for (int64_t c = 0; first + c < P; ++c) {
            float xf[1], gf[1];
            V1::widen(reinterpret_cast<mem1_t *>(x)[c], xf);
            V1::widen(reinterpret_cast<const mem1_t *>(g)[c], gf);
            xf[0] = fmaf(-gamma, gf[0], xf[0]);
            reinterpret_cast<mem1_t *>(x)[c] = V1::narrow(xf);
        }
    }
}
}  // namespace

hipError_t launch_local_step(void *X, int dtype, int64_t N, int64_t P, int64_t row_stride, const void *G,
                             int64_t g_row_stride, const uint8_t *alive, float gamma, hipStream_t stream)
{
    const int64_t esize = dtype == 0 ? 4 : 2, ve = 16 / esize;
    const int64_t tiles = (P + ve * 256 - 1) / (ve * 256);
    const int64_t blocks = tiles * N;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    char *x = static_cast<char *>(X);
    const char *g = static_cast<const char *>(G);
    const dim3 grid(static_cast<uint32_t>(blocks)), block(256);
    if (dtype == 0)
        local_step_kernel<0, 4><<<grid, block, 0, stream>>>(x, row_stride * esize, g, g_row_stride * esize, P, alive, gamma, tiles);
    else
        local_step_kernel<1, 8><<<grid, block, 0, stream>>>(x, row_stride * esize, g, g_row_stride * esize, P, alive, gamma, tiles);
    return hipGetLastError();
}

}  // namespace moshpit
