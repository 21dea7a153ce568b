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
    uint16_t bucket[kMax];      // of every peer; kAbsent = sits the round out
    uint16_t members[kMax];     // bucket by bucket
};
constexpr uint16_t kAbsent = 0xffff;

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
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    for (int32_t k = tid; k < n_buckets; k += kThreads) sh.count[k] = 0;
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
        sh.bucket[i] = mine[u] < 0 ? kAbsent : static_cast<uint16_t>(mine[u]);
        if (mine[u] >= 0) at[u] = atomicAdd(&sh.count[mine[u]], 1);
    }
    __syncthreads();

    // exclusive scans over the buckets: members, and groups of at most M
    int32_t c[kPer], sum = 0, groups = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int32_t k = tid * kPer + u;
        c[u] = k < n_buckets ? sh.count[k] : 0;
        sum += c[u];
        if constexpr (KEYED) groups += (c[u] + M - 1) / M;
    }
    int32_t before = sum, groups_before = groups;
#pragma unroll
    for (int32_t off = 1; off < 64; off <<= 1) {
        const int32_t a = __shfl_up(before, off, 64), b = __shfl_up(groups_before, off, 64);
        if (lane >= off) {
            before += a;
            groups_before += b;
        }
    }
    if (lane == 63) {
        sh.wave_sums[0][wave] = before;
        sh.wave_sums[1][wave] = groups_before;
    }
    __syncthreads();
    before -= sum;
    groups_before -= groups;
    for (int32_t w = 0; w < wave; ++w) {
        before += sh.wave_sums[0][w];
        groups_before += sh.wave_sums[1][w];
    }
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
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (mine[u] >= 0) sh.members[sh.start[mine[u]] + at[u]] = static_cast<uint16_t>(tid + u * kThreads);
    __syncthreads();

#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (mine[u] < 0) continue;
        const int32_t i = tid + u * kThreads, first = sh.start[mine[u]], n = sh.count[mine[u]];
        int32_t rank = 0;
        for (int32_t k = 0; k < n; ++k) {
            const int32_t j = sh.members[first + k];
            const uint64_t other = sh.order[j];
            rank += (other < key[u] || (other == key[u] && j < i)) ? 1 : 0;
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
