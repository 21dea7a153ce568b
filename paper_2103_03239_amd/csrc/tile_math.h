// Arithmetic of an averaging round on a tile that lies in LDS, for gfx950: how CV columns of a
// row are read and written, the balanced summation tree, lane exchanges and the division shared
// by several columns.  Used by the kernels that run several rounds on one tile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf16_round.h"
#include "grid_plan.h"
#include "row_vec.h"

namespace moshpit {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kNormalOrZero = 0x168;  // v_cmp_class mask: -normal, -0, +0, +normal

// Block barrier that orders LDS traffic only.  __syncthreads() also waits for
// every outstanding global load and store of the wave (its fence covers global
// memory), which would serialise the tile prefetch and the store drain with
// the rounds running in LDS.  Threads of a block exchange data through LDS
// only, so waiting for the LDS counter before the barrier is sufficient.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Lane exchanges without a trip through LDS.  With rows of 16 lanes r0..r3,
//   swap16(a, b) = ([a.r0, b.r0, a.r2, b.r2], [a.r1, b.r1, a.r3, b.r3])
//   swap32(a, b) = ([a.r0, a.r1, b.r0, b.r1], [a.r2, a.r3, b.r2, b.r3])
// (v_permlane16_swap / v_permlane32_swap).  Adding the two results of a swap of
// two DIFFERENT values reduces both across a pair of rows at once and leaves
// one of them in each row of the pair: the transposing reduction used below.
struct LanePair { float first, second; };
__device__ __forceinline__ LanePair swap16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair swap32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// The same of binary64 values.
struct DoublePair { double first, second; };
template <bool FAR> __device__ __forceinline__ DoublePair swap_halves(double a, double b)
{
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const uint32_t xl = static_cast<uint32_t>(x), xh = static_cast<uint32_t>(x >> 32), yl = static_cast<uint32_t>(y), yh = static_cast<uint32_t>(y >> 32);
    const auto l = FAR ? __builtin_amdgcn_permlane32_swap(xl, yl, false, false) : __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = FAR ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false) : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    return DoublePair{__builtin_bit_cast(double, static_cast<uint64_t>(h[0]) << 32 | l[0]), __builtin_bit_cast(double, static_cast<uint64_t>(h[1]) << 32 | l[1])};
}
template <int CTRL> __device__ __forceinline__ double rotated(double v)
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(bits), CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(bits >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}
// Sum over the lanes of a row of 16 that differ by multiples of 1 << from (every lane gets it), by rotations.
__device__ __forceinline__ double row_sum(double v, int32_t from)
{
    if (from <= 3) v += rotated<0x128>(v);
    if (from <= 2) v += rotated<0x124>(v);
    if (from <= 1) v += rotated<0x122>(v);
    if (from <= 0) v += rotated<0x121>(v);
    return v;
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = row_sum(v, 0);
    DoublePair p = swap_halves<false>(v, v);
    v = p.first + p.second;
    p = swap_halves<true>(v, v);
    return p.first + p.second;
}

// Distortion of a tile in LDS: sum over its columns of s2 - s1^2 / N, s1 and s2 the sums of the differences from one row
// and of their squares.  A lane holds s1 of the NE columns of its vector (lane & (vectors - 1)) and s2 of all of them
// together.  column_sums: those of a wave, to LDS: cols[NE << wv_shift], *squares.  The lanes that share a column are added by
// exchanges that halve the columns of a lane (a sum of four columns over four lanes takes 3 additions and 6
// exchanges instead of 8 and 16).
template <int NE> __device__ __forceinline__ void column_sums(const double (&s1)[NE], double s2, int32_t wv_shift, double *cols, double *squares)
{
    asm volatile("" : "+s"(wv_shift));           // (what is asked of it below is not kept in registers from round to round)
    const int32_t lane = threadIdx.x & 63;
    const double all = wave_sum(s2);
    if (lane == 0) *squares = all;
    double *mine = cols + (lane & ((1 << wv_shift) - 1)) * NE;
    if (wv_shift >= 6) {
#pragma unroll
        for (int e = 0; e < NE; ++e) mine[e] = s1[e];
        return;
    }
    double half[NE / 2];
#pragma unroll
    for (int e = 0; e < NE / 2; ++e) {
        const DoublePair p = swap_halves<true>(s1[e], s1[e + NE / 2]);      // lower half of the wave: column e
        half[e] = p.first + p.second;
    }
    mine += (lane >> 5) * (NE / 2);
    if (wv_shift == 5) {
#pragma unroll
        for (int e = 0; e < NE / 2; ++e) mine[e] = half[e];
        return;
    }
    double quarter[NE / 4];
#pragma unroll
    for (int e = 0; e < NE / 4; ++e) {
        const DoublePair p = swap_halves<false>(half[e], half[e + NE / 4]);  // rows 0 and 2: column e
        quarter[e] = row_sum(p.first + p.second, wv_shift);
    }
    mine += ((lane >> 4) & 1) * (NE / 4);
    if ((lane & 15) >> wv_shift == 0)
#pragma unroll
        for (int e = 0; e < NE / 4; ++e) mine[e] = quarter[e];
}
// One wave: the sum over the columns, from what `parts` parts of the rows left in cols and `waves` waves in squares; inv = 1 / n.
// (columns outside the tile hold 0)
__device__ __forceinline__ double finish_columns(const double *cols, int32_t parts, int32_t columns, const double *squares, int32_t waves, double n, double inv)
{
    const int32_t lane = threadIdx.x & 63;
    double sum = lane < waves ? squares[lane] : 0.0, t2 = 0.0;
    for (int32_t q = lane; q < columns; q += 64) {
        double t1 = 0.0;
#pragma unroll 4
        for (int32_t k = 0; k < parts; ++k) t1 += cols[k * columns + q];
        t2 = fma(t1, t1, t2);
    }
    return wave_sum(sum - over(t2, n, inv));            // (one quotient a lane)
}

// CV consecutive columns of one row in LDS, widened to binary32.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int DT, int CV> struct Cols;
template <> struct Cols<0, 4> {
    typedef float elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[4])
    {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(p);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[4])
    {
        *reinterpret_cast<f32x4 *>(p) = f32x4{f[0], f[1], f[2], f[3]};
    }
};
template <> struct Cols<0, 2> {
    typedef float elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[2])
    {
        const f32x2 v = *reinterpret_cast<const f32x2 *>(p);
        f[0] = v.x; f[1] = v.y;
    }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[2])
    {
        *reinterpret_cast<f32x2 *>(p) = f32x2{f[0], f[1]};
    }
};
template <> struct Cols<0, 1> {
    typedef float elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[1]) { f[0] = *p; }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[1]) { *p = f[0]; }
};
template <> struct Cols<1, 4> {
    typedef uint16_t elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[4])
    {
        const u32x2 v = *reinterpret_cast<const u32x2 *>(p);
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[4])
    {
        *reinterpret_cast<u32x2 *>(p) = u32x2{bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3])};
    }
};
template <> struct Cols<1, 2> {
    typedef uint16_t elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[2])
    {
        const uint32_t v = *reinterpret_cast<const uint32_t *>(p);
        f[0] = __uint_as_float(v << 16); f[1] = __uint_as_float(v & 0xffff0000u);
    }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[2])
    {
        *reinterpret_cast<uint32_t *>(p) = bf16_pair(f[0], f[1]);
    }
};
template <> struct Cols<1, 1> {
    typedef uint16_t elem_t;
    static __device__ __forceinline__ void load(const elem_t *p, float (&f)[1])
    {
        f[0] = __uint_as_float(static_cast<uint32_t>(*p) << 16);
    }
    static __device__ __forceinline__ void store(elem_t *p, const float (&f)[1])
    {
        *p = bf16_one(f[0]);
    }
};

// One 16-byte tile slot (4 binary32 or 8 bfloat16 values) after a local step of
// Moshpit SGD (Alg. 2): x - gamma * g, formed in binary32 with one fused multiply-add
// per value and rounded to the storage type.
template <int DT> __device__ __forceinline__ u32x4 local_step(const u32x4 &x, const u32x4 &g, float gamma)
{
    if constexpr (DT == 0) {
        u32x4 out;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[e] = __float_as_uint(__fmaf_rn(-gamma, __uint_as_float(g[e]), __uint_as_float(x[e])));
        return out;
    } else {
        u32x4 out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = __fmaf_rn(-gamma, __uint_as_float(g[e] << 16), __uint_as_float(x[e] << 16));
            const float hi = __fmaf_rn(-gamma, __uint_as_float(g[e] & 0xffff0000u), __uint_as_float(x[e] & 0xffff0000u));
            out[e] = bf16_pair(lo, hi);
        }
        return out;
    }
}

// Sum of TREE positions j0..j0+TREE-1 of CV columns of a group, as the balanced
// tree ((x0+x1)+(x2+x3))+...; positions whose bit is clear (absent peers, and
// positions past the group, whose bits are never set) contribute an exact 0:
// their read is redirected to `zeros`, 16 bytes of LDS that hold 0, which costs
// one select per position instead of one per value.  Blocks of up to FLAT
// positions are read at once; larger trees are the sum of their two balanced
// halves, which bounds the register footprint.
template <int DT, int CV, int TREE, int FLAT>
__device__ __forceinline__ void tree_block(const typename Cols<DT, CV>::elem_t *col, int32_t step, int32_t j0,
                                           const typename Cols<DT, CV>::elem_t *zeros, uint32_t bits,
                                           float (&out)[CV])
{
    if constexpr (TREE > FLAT) {
        float lo[CV], hi[CV];
        tree_block<DT, CV, TREE / 2, FLAT>(col, step, j0, zeros, bits & ((1u << (TREE / 2)) - 1u), lo);
        tree_block<DT, CV, TREE / 2, FLAT>(col, step, j0 + TREE / 2, zeros, bits >> (TREE / 2), hi);
#pragma unroll
        for (int e = 0; e < CV; ++e) out[e] = lo[e] + hi[e];
    } else {
        float f[TREE][CV];
#pragma unroll
        for (int u = 0; u < TREE; ++u) {
            const bool on = (bits >> u) & 1u;
            Cols<DT, CV>::load(on ? col + (j0 + u) * step : zeros, f[u]);
        }
#pragma unroll
        for (int s = 1; s < TREE; s *= 2)
#pragma unroll
            for (int u = 0; u + s < TREE; u += 2 * s)
#pragma unroll
                for (int e = 0; e < CV; ++e) f[u][e] += f[u + s][e];
#pragma unroll
        for (int e = 0; e < CV; ++e) out[e] = f[0][e];
    }
}

// acc / k for CV columns, sharing the reciprocal y = RN(1/k): q0 = RN(acc * y), the exact
// remainder r = acc - k * q0 (one fma), q = RN(q0 + r * y) is the correctly rounded quotient
// whenever nothing underflows.  A q that is not a normal number or zero (NaN from an infinite
// sum, subnormal) is redone with a true division.  With this guard the sequence was compared
// with the division for every count k <= 64 and all 2^32 binary32 numerators: the only
// difference is -0 / k, and acc is never -0 (it starts from +0).
template <int CV> __device__ __forceinline__ void divide_columns(float (&acc)[CV], float k, float y)
{
    float quo[CV];
    bool redo = false;
#pragma unroll
    for (int e = 0; e < CV; ++e) {
        const float q0 = __fmul_rn(acc[e], y);
        const float r = __fmaf_rn(-k, q0, acc[e]);
        quo[e] = __fmaf_rn(r, y, q0);
        redo = redo || !__builtin_amdgcn_classf(quo[e], kNormalOrZero);
    }
    if (redo) {
#pragma unroll
        for (int e = 0; e < CV; ++e) quo[e] = acc[e] / k;
    }
#pragma unroll
    for (int e = 0; e < CV; ++e) acc[e] = quo[e];
}

// SPLIT lanes (16 or 32 apart) of an item hold partial sums part[0..3] of its 4 columns.  They
// are added across lanes so that each lane ends with the total of ONE column (same order as the
// full tree: (s0 + s1) + (s2 + s3)), divides that one, and the quotients are handed round: 6 (4)
// exchanges and 1 (2) divisions per lane instead of 8 (4) exchanges and 4 divisions.
template <int SPLIT>
__device__ __forceinline__ void mean_over_lanes(const float (&part)[4], float k, float (&mean4)[4])
{
    static_assert(SPLIT == 2 || SPLIT == 4, "2 or 4 lanes share an item");
    if constexpr (SPLIT == 4) {
        const LanePair a = swap16(part[0], part[1]);    // rows 0, 2: column 0; rows 1, 3: column 1
        const LanePair b = swap16(part[2], part[3]);    // rows 0, 2: column 2; rows 1, 3: column 3
        const LanePair c = swap32(a.first + a.second, b.first + b.second);
        const float mean = (0.f + (c.first + c.second)) / k;    // row r: column r
        const LanePair eo = swap16(mean, mean);         // columns 0|2 and 1|3 of my half
        const LanePair m02 = swap32(eo.first, eo.first);
        const LanePair m13 = swap32(eo.second, eo.second);
        mean4[0] = m02.first; mean4[1] = m13.first; mean4[2] = m02.second; mean4[3] = m13.second;
    } else {
        const LanePair a = swap32(part[0], part[1]);    // lower half: column 0, upper: column 1
        const LanePair b = swap32(part[2], part[3]);    // lower half: column 2, upper: column 3
        const float q01 = (0.f + (a.first + a.second)) / k;
        const float q23 = (0.f + (b.first + b.second)) / k;
        const LanePair m01 = swap32(q01, q01);
        const LanePair m23 = swap32(q23, q23);
        mean4[0] = m01.first; mean4[1] = m01.second; mean4[2] = m23.first; mean4[3] = m23.second;
    }
}

}  // namespace moshpit
