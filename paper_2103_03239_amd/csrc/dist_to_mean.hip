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
// Mapping (dist_rows_kernel).  A block owns a tile of `lanes` vectors of 16 bytes of every row; a
// wave has 64 / lanes rows in one load, eight loads in flight and its block's waves take turns along the
// rows.  Their per-column sums meet across lanes and in LDS, and the block writes ONE partial.  A second
// one-block kernel adds the partials in a fixed order, so the result does not depend on scheduling.
//
// What bounds it (MI355X): HBM where there are enough tiles (6.3 to 6.9 TB/s from 1.6 GB on, 5.3 to 5.9 in the pass that follows a
// write, whose lines it pushes out of the last-level cache); below, the walk along the rows, so tiles get narrower until the chip has
// waves enough (dist_tiles.h).  A tile was 64 vectors wide whatever the state's shape, with a wave for 256 rows of it.  us, both kernels, repeated
// passes (the pass after a write), then and now:
//   1024 rows, 25 MB            binary32 26 -> 7.8 (34 -> 13)      bfloat16 52 -> 11 (56 -> 15)
//   256 rows, 6.4 MB            22 -> 7.1 (32 -> 10)               33 -> 8.2 (53 -> 12)
//   4096 rows, 100 MB           79 -> 19 (60 -> 23)                111 -> 22 (102 -> 25)
//   512 rows, 400 MB            64 -> 62 (73 -> 66)                100 -> 64 (95 -> 66)
//   4096 rows, 1.6 GB           266 -> 245 (311 -> 297)            291 -> 256 (327 -> 307)
//   4096 rows, 2.1 GB           350 -> 333 (414 -> 369)            353 -> 339 (384 -> 394)
//   16 rows, 1.6 GB             328 -> 245 (391 -> 305)            330 -> 245 (379 -> 303)
//   1024 rows, 17 GB            2,588 -> 2,497 (2,929 -> 2,910)
// dist_partial_kernel takes a row mask, and rows of less than 16 bytes.
#include <mutex>

#include "dist_tiles.h"
#include "moshpit_internal.h"
#include "row_vec.h"
#include "sum_partials.h"

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

constexpr int kRowLoads = 8;       // of a lane in flight
constexpr int kDieRun = 32;

// The same where every row counts and has 16 bytes or more.  LANES lanes of a wave take a row's part of the tile, the
// others the rows after it.  Dynamic LDS: rows_lds_bytes (sized by the block's waves: one-wave blocks take none, with
// the 33 KB of 16 waves five of them shared a compute unit, and 16 rows of 100 MB took 425 us instead of 243).
constexpr int rows_lds_bytes(int lanes, int waves) { return waves == 1 ? 0 : (4 * lanes + 1) * waves * 8; }

template <int DT, int LANES, bool NT>
__global__ __launch_bounds__(8 * 64, 4) void dist_rows_kernel(const char *__restrict__ X, int64_t row_bytes, int64_t valid_bytes,
                                                           int32_t N, bool last_first, double *__restrict__ partials)
{
    typedef Wide<DT, DT == 0 ? 4 : 8> V;
    typedef typename V::mem_t mem_t;
    constexpr int NE = V::NE, kRows = 64 / LANES;
    extern __shared__ __align__(16) double lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int c = lane & (LANES - 1), sub = lane / LANES;
    // Blocks b, b + 8, b + 16, ... run on the same one of the 8 dies; each die takes kDieRun neighbouring tiles, so that
    // the parts of a cache line that two of them share meet in its L2.
    int64_t tile = blockIdx.x;
    const int64_t span = tile / (8 * kDieRun) * (8 * kDieRun), in_span = tile - span;
    if (span + 8 * kDieRun <= gridDim.x) tile = span + (in_span & 7) * kDieRun + (in_span >> 3);
    const int64_t begin = (tile * LANES + c) * 16;
    const bool valid = begin < valid_bytes;                 // (a lane past the row reads its last vector, for nothing)
    const int64_t at = begin < valid_bytes - 16 ? begin : valid_bytes - 16;
    const int shared = static_cast<int>((begin - at) / (16 / NE));           // elements that belong to the neighbour
    const char *col = X + at;

    double x0[NE], s1[NE], s2[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) { s1[e] = 0.0; s2[e] = 0.0; }
    V::widen(load_vec<false, mem_t>(col), x0);
    const auto add = [&](const mem_t &row) {
        double x[NE];
        V::widen(row, x);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const double dlt = x[e] - x0[e];
            s1[e] += dlt;
            s2[e] = fma(dlt, dlt, s2[e]);
        }
        if constexpr (NE == 8) __builtin_amdgcn_sched_barrier(0);       // (two rows' doubles at once spill)
    };
    // From the last row to the first (see dist_tiles.h) or from the first to the last: row 0 is the one that is subtracted either way.
    const int32_t step = waves * kRows, start = wave * kRows + sub;
    const int64_t step_bytes = last_first ? -(step * row_bytes) : step * row_bytes;
    const char *from = col + (last_first ? N - 1 - start : start) * row_bytes;
    int32_t i = wave * kRows;                               // rows taken before the wave's next load
    for (; i + (kRowLoads - 1) * step + kRows <= N; i += kRowLoads * step) {
        mem_t buf[kRowLoads];
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            buf[u] = load_vec<NT, mem_t>(from);
            from += step_bytes;
        }
        // All loads leave before the first row is added: the compiler's own order keeps fewer in flight (256 rows of 2.6 GB
        // bfloat16, tiles of 64 lanes and 8 waves, 416 -> 373 us; 4096 rows of 2.9 GB 483 -> 425).
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) add(buf[u]);
    }
    if (i < N) {
        // (row 0, whose difference is 0, in the place of rows that there are not)
        mem_t buf[kRowLoads];
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            buf[u] = load_vec<NT, mem_t>(i + u * step + sub < N ? from : col);
            from += step_bytes;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) add(buf[u]);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int off = 32; off >= LANES; off >>= 1) {
            s1[e] += __shfl_xor(s1[e], off, 64);
            s2[e] += __shfl_xor(s2[e], off, 64);
        }

    double mine = 0.0;
    if (waves == 1) {
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (valid && sub == 0 && e >= shared) mine += s2[e] - s1[e] * s1[e] / static_cast<double>(N);
    } else {
        // the waves' sums of element e of every vector meet in one of two buffers, and wave e % waves adds them
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            double *here = lds + (e & 1) * 2 * waves * LANES;
            if (sub == 0) {
                here[wave * LANES + c] = s1[e];
                here[(waves + wave) * LANES + c] = s2[e];
            }
            __syncthreads();
            if (wave == (e & (waves - 1)) && sub == 0) {
                double t1 = 0.0, t2 = 0.0;
                for (int w = 0; w < waves; ++w) { t1 += here[w * LANES + c]; t2 += here[(waves + w) * LANES + c]; }
                if (valid && e >= shared) mine += t2 - t1 * t1 / static_cast<double>(N);
            }
        }
    }
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1) mine += __shfl_down(mine, off, 64);
    if (waves == 1) {
        if (lane == 0) partials[blockIdx.x] = mine;
        return;
    }
    double *total = lds + 4 * waves * LANES;
    if (lane == 0) total[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int w = 0; w < waves; ++w) sum += total[w];
        partials[blockIdx.x] = sum;
    }
}

__global__ __launch_bounds__(kSumThreads) void dist_final_kernel(const double *__restrict__ partials, int64_t count,
                                                                 int64_t n, double *__restrict__ out)
{
    const double sum = block_sum(partials, count);
    if (threadIdx.x == 0) out[0] = sum / static_cast<double>(n);
}

// Blocks of dist_partial_kernel.
int64_t general_blocks(int dtype, int64_t P)
{
    const int64_t valid_bytes = P * (dtype == 0 ? 4 : 2);
    const int64_t nvec = valid_bytes < 16 ? P : (valid_bytes + 15) / 16;
    return (nvec + 63) / 64;
}

template <int DT, int LANES>
hipError_t launch_rows(const char *X, int64_t row_bytes, int64_t valid_bytes, int64_t N, const DistTiles &t, double *partials,
                       hipStream_t stream)
{
    const auto kernel = t.streaming ? dist_rows_kernel<DT, LANES, true> : dist_rows_kernel<DT, LANES, false>;
    kernel<<<dim3(static_cast<uint32_t>(t.blocks)), dim3(t.waves * 64), rows_lds_bytes(LANES, t.waves), stream>>>(
        X, row_bytes, valid_bytes, static_cast<int32_t>(N), t.last_first, partials);
    return hipGetLastError();
}
template <int DT>
hipError_t launch_rows_of(const char *X, int64_t row_bytes, int64_t valid_bytes, int64_t N, const DistTiles &t, double *partials,
                          hipStream_t stream)
{
    switch (t.lanes) {
    case 64: return launch_rows<DT, 64>(X, row_bytes, valid_bytes, N, t, partials, stream);
    case 32: return launch_rows<DT, 32>(X, row_bytes, valid_bytes, N, t, partials, stream);
    case 16: return launch_rows<DT, 16>(X, row_bytes, valid_bytes, N, t, partials, stream);
    case 8: return launch_rows<DT, 8>(X, row_bytes, valid_bytes, N, t, partials, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

int64_t dist_partials_count(int dtype, int64_t N, int64_t P)
{
    int64_t most = general_blocks(dtype, P);
    for (int whole_lines = 0; whole_lines < 2; ++whole_lines) {
        DistTiles t;
        if (dist_tiles(dtype == 0 ? 4 : 2, N, P, whole_lines != 0, &t) && t.blocks > most) most = t.blocks;
    }
    return most;
}

hipError_t launch_dist_to_mean(const void *X, int dtype, int64_t N, int64_t P, int64_t row_stride,
                               double *partials, double *out, const uint8_t *present, int64_t first, int64_t n,
                               hipStream_t stream)
{
    const int64_t esize = dtype == 0 ? 4 : 2;
    const int64_t row_bytes = row_stride * esize, valid_bytes = P * esize;
    const char *base = static_cast<const char *>(X);
    DistTiles tiles;
    int64_t blocks = 0;
    hipError_t e = hipSuccess;
    const bool whole_lines = reinterpret_cast<uintptr_t>(X) % 128 == 0 && row_bytes % 128 == 0;
    if (present == nullptr && dist_tiles(esize, N, P, whole_lines, &tiles)) {
        blocks = tiles.blocks;
        e = dtype == 0 ? launch_rows_of<0>(base, row_bytes, valid_bytes, N, tiles, partials, stream)
                       : launch_rows_of<1>(base, row_bytes, valid_bytes, N, tiles, partials, stream);
    } else {
        blocks = general_blocks(dtype, P);
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        // about 256 rows per wave
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
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    dist_final_kernel<<<dim3(1), dim3(sum_threads(blocks)), 0, stream>>>(partials, blocks, n, out);
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
