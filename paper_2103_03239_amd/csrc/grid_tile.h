// What the kernels that run several rounds on a whole grid have in common (grid_rounds.hip,
// mean_rounds.hip): how the state is cut into tiles of all rows, which block takes which tile, and
// who is present in a round of a failure schedule.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mix64.h"
#include "moshpit_internal.h"
#include "row_vec.h"

namespace moshpit {

template <int DT> __device__ __forceinline__ void widen16(const u32x4 &m, float (&f)[DT == 0 ? 4 : 8])
{
    if constexpr (DT == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(m[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f[2 * e] = __uint_as_float(m[e] << 16);
            f[2 * e + 1] = __uint_as_float(m[e] & 0xffff0000u);
        }
    }
}

// n / d for n < 2^16 and magic = ceil(2^32 / d), d >= 2
__device__ __forceinline__ int32_t quotient(int32_t n, uint32_t magic)
{
    return static_cast<int32_t>(__umulhi(static_cast<uint32_t>(n), magic));
}

struct TileSpan {
    int64_t col0;          // first byte of the tile within a row
    int32_t seg;           // bytes of every row in it (>= 16)
};

// Tile w covers bytes [w * Wb, (w + 1) * Wb) of every row.  A last tile of fewer than 16 bytes
// takes the last vector of its neighbour as well.
__device__ __forceinline__ TileSpan tile_span(const GridPlan &p, int64_t w)
{
    TileSpan t;
    const int64_t left = p.valid_bytes - w * p.Wb;
    t.col0 = w * p.Wb;
    t.seg = static_cast<int32_t>(left < p.Wb ? left : p.Wb);
    if (t.seg < 16) {
        t.col0 -= 16;
        t.seg += 16;
    } else if (left > p.Wb && left < p.Wb + 16) {
        t.seg -= 16;
    }
    return t;
}

// Position i of the work list -> tile.  Blocks b, b + 8, b + 16, ... run on the same one of the 8
// dies; each die takes `run` consecutive tiles of every 8 * run, so that tiles that share cache
// lines or DRAM pages meet in one die's L2.  A copy of 4096 rows x 32 bytes moves 1.4 TB/s dealt in
// order, 3.7 TB/s in runs of 32 (ordinary loads and stores: they have to stay in L2; 1.3 TB/s with
// non-temporal ones).
__device__ __forceinline__ int64_t tile_of(const GridPlan &p, int64_t i)
{
    if (p.die_run <= 1) return i;
    const int64_t span = 8 * static_cast<int64_t>(p.die_run);
    const int64_t q = i / span;
    if ((q + 1) * span > p.tiles) return i;
    const int64_t r = i - q * span;
    return q * span + (r & 7) * p.die_run + (r >> 3);
}

// ---- who takes part ------------------------------------------------------------------------

constexpr int kPlanThreads = 1024;
constexpr int kPerThread = kGridMaxPeers / kPlanThreads;

__device__ __forceinline__ bool failure_event(uint64_t seed, int64_t s, int64_t i, uint32_t threshold)
{
    const uint64_t round_key = mix64(seed + 0x9E3779B97F4A7C15ull * static_cast<uint64_t>(s + 1));
    return static_cast<uint32_t>(mix64(round_key ^ static_cast<uint64_t>(i)) >> 40) < threshold;
}

// Is peer i present in round t0 + r (and in the round before it, if that belongs to the run)?
__device__ __forceinline__ void presence(const GridSchedule &s, int32_t i, int64_t r, bool &before, bool &now)
{
    before = true;
    const bool earlier = r > 0 || s.continued;
    if (s.masks != nullptr) {
        now = s.masks[r * s.N + i] != 0;
        if (earlier) before = s.masks[(r - 1) * s.N + i] != 0;
    } else {
        now = !failure_event(s.seed, s.t0 + r, i, s.threshold);
        if (s.refresh && earlier) before = !failure_event(s.seed, s.t0 + r - 1, i, s.threshold);
    }
}

}  // namespace moshpit
