// Average distortion (1/N) sum_i ||theta_i - theta_bar||^2, theta_bar the mean
// over all N rows (left-hand side of the equation of Thm 3.2; the error
// measure of Sec. 4.1), for gfx950.
//
// The state is read exactly once.  For every column c the kernel accumulates,
// in binary64, s1 = sum_i (x_ic - x_0c) and s2 = sum_i (x_ic - x_0c)^2 and uses
// sum_i (x_ic - mean_c)^2 = s2 - s1^2 / N.  Shifting by row 0 keeps the
// subtraction harmless once the peers have (nearly) agreed: all differences
// are then tiny and exact in binary64.  With a `present` mask (a partly filled
// grid) the same runs over the rows that hold a peer, shifted by the first one.
//
// Mapping.  A block owns a tile of 64 vectors (one 128-bit vector per lane,
// 1 KiB per row); its W waves (W chosen so that a wave sees about 256 rows) take
// rows w, w+W, ... with 8 (bfloat16: 4) non-temporal row loads in flight each, then
// combine their per-column sums through LDS, reduce across lanes and write ONE
// partial per block.  A second one-block kernel adds the partials in a fixed
// order, so the result does not depend on scheduling.
//
// What bounds it (MI355X).  Large states HBM: 1024 rows of 16 MiB at 6.9 TB/s.
// Short rows the walk of a wave over its 256 rows: 1024 rows of 15,625 binary32,
// 64 MB in 62 blocks, 67 us.  That walk took 146 us while every load stood behind
// a branch of its own, which made the compiler wait for it before the next; rows
// off the 16-byte boundaries, element by element in four times as many blocks, 71.
#include <mutex>

#include "moshpit_internal.h"
#include "row_vec.h"

// Partial sums of the allocation-free entry point: one double per block of the
// first kernel, kept in the code object so that no call ever allocates.  Every
// GPU the library runs on holds its own copy (1 MiB) at its own address until
// the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the kernels get the address that call returns.
static __device__ __align__(256) double scratch[moshpit::kStaticPartials];

namespace moshpit {
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[kMaxDevices] = {};     // device address of `scratch`, per device

constexpr int kMaxWaves = 16;      // waves per block: 1, 2, 4, 8 or 16

template <int DT, int VE> struct Wide;

template <> struct Wide<0, 4> {
    typedef f32x4 mem_t;
    static constexpr int NE = 4;
    static __device__ __forceinline__ void widen(const mem_t &m, double (&f)[NE])
    {
        f[0] = m.x; f[1] = m.y; f[2] = m.z; f[3] = m.w;
    }
};
template <> struct Wide<0, 1> {
    typedef float mem_t;
    static constexpr int NE = 1;
    static __device__ __forceinline__ void widen(const mem_t &m, double (&f)[NE]) { f[0] = m; }
};
template <> struct Wide<1, 8> {
    typedef u32x4 mem_t;
    static constexpr int NE = 8;
    static __device__ __forceinline__ void widen(const mem_t &m, double (&f)[NE])
    {
        const uint32_t w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f[2 * k] = __uint_as_float(w[k] << 16);
            f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
        }
    }
};
template <> struct Wide<1, 1> {
    typedef uint16_t mem_t;
    static constexpr int NE = 1;
    static __device__ __forceinline__ void widen(const mem_t &m, double (&f)[NE])
    {
        f[0] = __uint_as_float(static_cast<uint32_t>(m) << 16);
    }
};

// X         byte pointer to element (row 0, first column of this launch)
// valid_bytes  bytes of a row; it has ceil(valid_bytes / vector size) vectors of VE elements.
//           Rows may start on any element; where a row is not a whole number of vectors its last
//           one ends with the row and the elements it shares with its neighbour count as 0 in it.
// partials  one double per block: sum over the block's columns of s2 - s1^2/n
// present   nullptr, or N bytes: rows with 0 are left out of mean and sum
//           (vertices of a partly filled grid that hold no peer)
// first     index of the first row that counts; n = number of rows that count
template <int DT, int VE, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void dist_partial_kernel(const char *__restrict__ X, int64_t row_bytes,
                                                                    int64_t valid_bytes, int64_t N,
                                                                    double *__restrict__ partials,
                                                                    const uint8_t *__restrict__ present,
                                                                    int64_t first, int64_t n)
{
    typedef Wide<DT, VE> V;
    typedef typename V::mem_t mem_t;
    constexpr int NE = V::NE;
    __shared__ double sh[2][kWaves][64];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t v = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    constexpr int64_t kVec = sizeof(mem_t);
    const bool valid = v * kVec < valid_bytes;            // (a lane past the row reads its last vector, for nothing)
    const int64_t at = v * kVec < valid_bytes - kVec ? v * kVec : valid_bytes - kVec;
    const int shared = static_cast<int>((v * kVec - at) / (kVec / NE));      // elements that belong to the neighbour
    const char *col = X + at;

    constexpr int kRowsInFlight = NE == 8 ? 4 : 8;           // (16 sums of 8 values leave registers for 4)
    double x0[NE], s1[NE], s2[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) { x0[e] = 0.0; s1[e] = 0.0; s2[e] = 0.0; }
    V::widen(load_vec<false, mem_t>(col + first * row_bytes), x0);
    // The wave looks at 64 of its rows at a time, then takes those that count, kRowsInFlight of them at once.
    // Where fewer are left the others are row `first`, whose difference is 0: without a branch around
    // them all the loads are issued before the first is used.
    for (int64_t i0 = __builtin_amdgcn_readfirstlane(wave); i0 < N; i0 += kWaves * 64) {
        const int64_t mine = i0 + static_cast<int64_t>(lane) * kWaves;
        uint64_t rows = __ballot(mine < N && (present == nullptr || present[mine] != 0));
        while (rows != 0) {
            mem_t buf[kRowsInFlight];
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u) {
                const int64_t i = rows != 0 ? i0 + static_cast<int64_t>(__builtin_ctzll(rows)) * kWaves : first;
                rows &= rows - 1;
                buf[u] = load_vec<true, mem_t>(col + i * row_bytes);
            }
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u) {
                double x[NE];
                V::widen(buf[u], x);
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    const double dlt = x[e] - x0[e];
                    s1[e] += dlt;
                    s2[e] = fma(dlt, dlt, s2[e]);
                }
            }
        }
    }

    // combine the waves' per-column sums, one element of the vector at a time
    double colsum = 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        sh[0][wave][lane] = s1[e];
        sh[1][wave][lane] = s2[e];
        __syncthreads();
        if (wave == 0) {
            double t1 = 0.0, t2 = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) { t1 += sh[0][w][lane]; t2 += sh[1][w][lane]; }
            if (valid && e >= shared) colsum += t2 - t1 * t1 / static_cast<double>(n);
        }
        __syncthreads();
    }
    if (wave == 0) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) colsum += __shfl_down(colsum, off, 64);
        if (lane == 0) partials[blockIdx.x] = colsum;
    }
}

__global__ __launch_bounds__(256) void dist_final_kernel(const double *__restrict__ partials, int64_t count,
                                                         int64_t n, double *__restrict__ out)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += 256) acc += partials[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0] / static_cast<double>(n);
}

int64_t row_blocks(int dtype, int64_t P)
{
    const int64_t valid_bytes = P * (dtype == 0 ? 4 : 2);
    const int64_t nvec = valid_bytes < 16 ? P : (valid_bytes + 15) / 16;
    return (nvec + 63) / 64;
}

}  // namespace

int64_t dist_partials_count(int dtype, int64_t P) { return row_blocks(dtype, P); }

hipError_t launch_dist_to_mean(const void *X, int dtype, int64_t N, int64_t P, int64_t row_stride,
                               double *partials, double *out, const uint8_t *present, int64_t first, int64_t n,
                               hipStream_t stream)
{
    const int64_t blocks = row_blocks(dtype, P);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const int64_t esize = dtype == 0 ? 4 : 2;
    const int64_t row_bytes = row_stride * esize, valid_bytes = P * esize;
    const char *base = static_cast<const char *>(X);
    // about 256 rows per wave (measured best on MI355X for 64 <= N <= 4096)
    int waves = 1;
    while (waves < kMaxWaves && N / (waves * 2) >= 256) waves *= 2;
    const dim3 grid(static_cast<uint32_t>(blocks));
#define MOSHPIT_DIST_CALL(DT, VE, W) \
    dist_partial_kernel<DT, VE, W><<<grid, dim3(W * 64), 0, stream>>>(base, row_bytes, valid_bytes, N, partials, present, first, n)
#define MOSHPIT_DIST(W)                                                                                        \
    if (waves == W) {                                                                                          \
        if (valid_bytes >= 16) {                                                                               \
            if (dtype == 0) MOSHPIT_DIST_CALL(0, 4, W);                                                        \
            else MOSHPIT_DIST_CALL(1, 8, W);                                                                   \
        } else {                                                                                               \
            if (dtype == 0) MOSHPIT_DIST_CALL(0, 1, W);                                                        \
            else MOSHPIT_DIST_CALL(1, 1, W);                                                                   \
        }                                                                                                      \
    }
    MOSHPIT_DIST(1)
    MOSHPIT_DIST(2)
    MOSHPIT_DIST(4)
    MOSHPIT_DIST(8)
    MOSHPIT_DIST(16)
#undef MOSHPIT_DIST
#undef MOSHPIT_DIST_CALL
    {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    dist_final_kernel<<<dim3(1), dim3(256), 0, stream>>>(partials, blocks, n, out);
    return hipGetLastError();
}

hipError_t static_scratch(double **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (ptr == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<double *>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace moshpit
