// The random orders of rounds whose groups are drawn anew, for up to 4096 peers, for gfx950: the
// permutation of Thm 3.2's scheme (App. C.3) and the order of peers_t behind the chunk indices of
// Alg. 1.  One launch of one block does the whole integer side of a round in LDS.
//
// Items are ranked by counting, not sorted: a first key with a small range puts every peer into a
// bucket (LDS atomics, then one scan over the buckets), and its rank within the bucket is the
// number of members with a smaller (order key, index).  The buckets are the chunk-index keys, or
// the upper 12 bits of the uniform order keys, so they hold about M peers, or one.  The result does
// not depend on the order in which the atomics land.
//
// Chunk-index keys can come together (a round in which a peer is alone in its group gives it chunk
// 0), up to all 4096 peers in one bucket.  Counting within it is quadratic (926 us a round), so as
// soon as a bucket holds more than kCrowded peers the members of every bucket are first spread
// over as many slots as it has members, by their uniform order keys, and counted within a slot.
//
// What bounds it: latency, about a dozen barriers.  The general path (dynamic_keys.hip,
// schedule.hip: a bitonic network over 4096 items and five more launches) takes 85 us a round at
// 4096 peers, this 12 us.
#include "mix64.h"
#include "moshpit_internal.h"

namespace moshpit {
namespace {

constexpr int kThreads = 1024;
constexpr int kMax = kSmallOrderPeers;
constexpr int kPer = kMax / kThreads;

struct Shared {
    uint64_t order[kMax];
    int32_t count[kMax];
    int32_t start[kMax];        // first position of the bucket
    int32_t group[kMax];        // first group of the bucket (chunk-index rounds)
    int32_t wave_sums[2][kThreads / 64];
    int32_t crowded;            // some bucket holds more than kCrowded
    alignas(16) uint16_t members[kMax];     // bucket by bucket (slot by slot); read eight at a time
    int32_t slot[kMax + 1];     // crowded rounds: members of a slot, then its first position; the slots of a
                                // bucket lie where its members do
};
// (well above the members of a bucket whose keys are spread, at most 64 where everybody takes part: 64 x
// 64 peers 36 us a round with 64 to a bucket, 38 with 2048 in one)
constexpr int32_t kCrowded = 128;

// Exclusive sums over the block of two values per thread.
__device__ __forceinline__ void block_scan(Shared &sh, int32_t &a, int32_t &b)
{
    const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t own_a = a, own_b = b;
#pragma unroll
    for (int32_t off = 1; off < 64; off <<= 1) {
        const int32_t x = __shfl_up(a, off, 64), y = __shfl_up(b, off, 64);
        if (lane >= off) {
            a += x;
            b += y;
        }
    }
    if (lane == 63) {
        sh.wave_sums[0][wave] = a;
        sh.wave_sums[1][wave] = b;
    }
    __syncthreads();
    a -= own_a;
    b -= own_b;
    for (int32_t w = 0; w < wave; ++w) {
        a += sh.wave_sums[0][w];
        b += sh.wave_sums[1][w];
    }
}

// KEYED: chunk-index round (buckets = keys, list padded per key, keys shifted).  Otherwise the
// permutation: index[rank] = peer, -1 where the mask leaves the peer out.
template <bool KEYED>
__global__ __launch_bounds__(kThreads) void small_order_kernel(int32_t N, int32_t M, int32_t kd, uint64_t seed, int64_t t,
                                                               int32_t masked, PeerBits bits, int32_t n_buckets,
                                                               int32_t *__restrict__ keys, int32_t *__restrict__ index,
                                                               int32_t n_index)
{
    extern __shared__ __align__(16) char lds[];
    Shared &sh = *reinterpret_cast<Shared *>(lds);
    const int32_t tid = threadIdx.x;

    for (int32_t k = tid; k < n_buckets; k += kThreads) sh.count[k] = 0;
    if (tid == 0) sh.crowded = 0;
    if constexpr (KEYED)
        for (int32_t k = tid; k < n_index; k += kThreads) index[k] = -1;
    __syncthreads();

    const uint64_t round_key = mix64(seed + 0xD1B54A32D192ED03ull * static_cast<uint64_t>(t + 1));
    int32_t mine[kPer], at[kPer];
    uint64_t key[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int32_t i = tid + u * kThreads;
        mine[u] = -1;
        at[u] = 0;
        key[u] = 0;
        if (i >= N) continue;
        const bool present = masked == 0 || ((bits.word[i >> 5] >> (i & 31)) & 1u) != 0;
        key[u] = mix64(round_key ^ static_cast<uint64_t>(i));
        if constexpr (KEYED) {
            if (present) {
                int32_t pk = 0, weight = 1;
                for (int32_t q = 0; q < kd; ++q) {
                    pk += keys[i * kd + q] * weight;
                    weight *= M;
                }
                mine[u] = pk;
            }
        } else {
            mine[u] = static_cast<int32_t>(key[u] >> 52);
        }
        sh.order[i] = key[u];
        if (mine[u] >= 0) at[u] = atomicAdd(&sh.count[mine[u]], 1);
        if (KEYED && at[u] == kCrowded) sh.crowded = 1;
    }
    __syncthreads();

    // exclusive scans over the buckets: members, and groups of at most M
    int32_t c[kPer], sum = 0, groups = 0;
    const bool crowded = KEYED && __builtin_amdgcn_readfirstlane(sh.crowded) != 0;    // the same for the whole block
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int32_t k = tid * kPer + u;
        c[u] = k < n_buckets ? sh.count[k] : 0;
        sum += c[u];
        if constexpr (KEYED) groups += (c[u] + M - 1) / M;
    }
    int32_t before = sum, groups_before = groups;
    block_scan(sh, before, groups_before);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int32_t k = tid * kPer + u;
        if (k < n_buckets) {
            sh.start[k] = before;
            sh.group[k] = groups_before;
        }
        before += c[u];
        if constexpr (KEYED) groups_before += (c[u] + M - 1) / M;
    }
    __syncthreads();
    int32_t spread[kPer];
    if (crowded) {
        for (int32_t k = tid; k <= kMax; k += kThreads) sh.slot[k] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            spread[u] = 0;
            if (mine[u] < 0) continue;
            // (key >> 32) / 2^32 of the way through the bucket, rounded down: ascending with the key
            spread[u] = sh.start[mine[u]] + static_cast<int32_t>(__umulhi(static_cast<uint32_t>(key[u] >> 32),
                                                                          static_cast<uint32_t>(sh.count[mine[u]])));
            at[u] = atomicAdd(&sh.slot[spread[u]], 1);
        }
        __syncthreads();
        int32_t n[kPer], first = 0, unused = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            n[u] = sh.slot[tid * kPer + u];
            first += n[u];
        }
        block_scan(sh, first, unused);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            sh.slot[tid * kPer + u] = first;
            first += n[u];
        }
        if (tid == kThreads - 1) sh.slot[kMax] = first;
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (mine[u] >= 0)
            sh.members[(crowded ? sh.slot[spread[u]] : sh.start[mine[u]]) + at[u]] = static_cast<uint16_t>(tid + u * kThreads);
    __syncthreads();

#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (mine[u] < 0) continue;
        const int32_t i = tid + u * kThreads, first = sh.start[mine[u]];
        int32_t rank = 0;
        if (crowded) {
            const int32_t begin = sh.slot[spread[u]], end = sh.slot[spread[u] + 1];
            rank = begin - first;
#pragma unroll 1
            for (int32_t k = begin; k < end; ++k) {                 // (one or two of them)
                const int32_t j = sh.members[k];
                const uint64_t other = sh.order[j];
                rank += (other < key[u] || (other == key[u] && j < i)) ? 1 : 0;
            }
        } else {
            const int32_t n = sh.count[mine[u]];
            for (int32_t k = 0; k < n; ++k) {
                const int32_t j = sh.members[first + k];
                const uint64_t other = sh.order[j];
                rank += (other < key[u] || (other == key[u] && j < i)) ? 1 : 0;
            }
        }
        if constexpr (KEYED) {
            const int32_t chunk = rank % M;                         // c_i: position within its group of at most M
            index[(sh.group[mine[u]] + rank / M) * M + chunk] = i;
            if (kd > 0) {
                for (int32_t q = 0; q + 1 < kd; ++q) keys[i * kd + q] = keys[i * kd + q + 1];
                keys[i * kd + kd - 1] = chunk;
            }
        } else {
            const bool present = masked == 0 || ((bits.word[i >> 5] >> (i & 31)) & 1u) != 0;
            index[first + rank] = present ? i : -1;
        }
    }
}

}  // namespace

hipError_t launch_small_permutation(uint64_t seed, int64_t t, int64_t N, const PeerBits *bits, int32_t *perm,
                                    hipStream_t stream)
{
    if (N <= 0 || N > kMax) return hipErrorInvalidValue;
    const auto kernel = small_order_kernel<false>;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), sizeof(Shared));
    if (e != hipSuccess) return e;
    kernel<<<dim3(1), dim3(kThreads), sizeof(Shared), stream>>>(static_cast<int32_t>(N), 1, 0, seed, t, bits != nullptr,
                                                                bits != nullptr ? *bits : PeerBits{}, kMax, nullptr, perm, 0);
    return hipGetLastError();
}

hipError_t launch_small_grouping(int64_t N, int32_t M, int32_t d, uint64_t seed, int64_t t, const PeerBits *bits,
                                 int32_t *keys, int32_t *index, int64_t n_index, hipStream_t stream)
{
    int64_t n_keys = 1;
    for (int32_t q = 0; q + 1 < d; ++q) n_keys *= M;
    if (N <= 0 || N > kMax || n_keys > kMax || n_index > 0x7fffffffLL) return hipErrorInvalidValue;
    const auto kernel = small_order_kernel<true>;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), sizeof(Shared));
    if (e != hipSuccess) return e;
    kernel<<<dim3(1), dim3(kThreads), sizeof(Shared), stream>>>(static_cast<int32_t>(N), M, d - 1, seed, t, bits != nullptr,
                                                                bits != nullptr ? *bits : PeerBits{},
                                                                static_cast<int32_t>(n_keys), keys, index,
                                                                static_cast<int32_t>(n_index));
    return hipGetLastError();
}

}  // namespace moshpit
