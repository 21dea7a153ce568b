// The random orders of rounds whose groups are drawn anew, for up to 4096 peers, for gfx950: the
// permutation of Thm 3.2's scheme (App. C.3) and the order of peers_t behind the chunk indices of
// Alg. 1.  One launch of one block does the whole integer side of a round in LDS.
//
// Items are ranked by counting, not sorted: peers fall into about as many buckets as there are peers,
// ascending by (chunk-index key, upper bits of the uniform order key) (LDS atomics, then one scan over the
// buckets), and a peer's rank within its bucket is the number of members with a smaller order key: one or two
// comparisons.  Order keys are a bijection of the index, so no two are equal, and the result does not
// depend on the order in which the atomics land.
//
// Chunk-index keys can come together (a round in which a peer is alone in its group gives it chunk
// 0), up to all 4096 peers with one key.  Counting within a bucket is quadratic, so as soon as one holds more
// than kCrowded peers the members of every bucket are first spread over as many slots as it has members, by
// the next bits of their order keys, and counted within a slot.
//
// What bounds it: latency of one block: the launch, one load of the keys, seven barriers.  In a launch of 1024 threads
// whatever the number of peers, buckets of about M peers each, keys loaded one after the other and the list
// written peer by peer, it took 19.4 us for 4096 peers; now 9.9.
// The general path (dynamic_keys.hip, schedule.hip: a bitonic network over 4096 items and five more launches) takes
// 85 us a round at 4096 peers.
#include "mix64.h"
#include "moshpit_internal.h"
#include "tile_math.h"

namespace moshpit {
namespace {

constexpr int kThreads = 1024;       // at most
static_assert(kThreads == kFewPeers, "a peer to a thread: the short argument block");
// Spreading costs 4096 peers 1.1 us a launch, 1024 0.8, counting 0.19 and 0.06 for every peer of the fullest bucket.  us, counted : spread: 4096
// peers, fullest bucket 8 10.4 : 11.5, 13 12.0 : 11.6, 24 13.9 : 11.8, 64 (64 x 64 peers with one key) 26 : 12, 256 64 : 12; 1024 peers 4 6.7 :
// 7.5, 20 7.4 : 7.5, 40 8.4 : 7.5, 500 31 : 8.  Where everybody takes part and keys are apart the fullest holds 8.
constexpr int32_t kCrowded = 16;

// Up to MAX peers, in up to MAX buckets.
template <int MAX> struct Shared {
    uint64_t order[MAX];                // order keys, bucket by bucket (slot by slot)
    int32_t count[MAX];
    int32_t start[MAX + 1];             // first position of the bucket
    int32_t group[MAX];                 // first group of the chunk-index key
    int32_t slot[MAX + 1];              // crowded rounds: members of a slot, then its first position; the slots of a
                                        // bucket lie where its members do
    int32_t wave_sums[3][kThreads / 64];
    int32_t crowded;                    // some bucket holds more than kCrowded
    alignas(16) uint16_t list[2 * MAX]; // the peer list (kNobody: nobody)
};
constexpr uint32_t kNobody = 0xffff;

template <int CTRL, int ROWS> __device__ __forceinline__ int32_t lanes_below(int32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
// Sum of the lanes up to this one; of its row of 16 only, without the last two steps.
__device__ __forceinline__ int32_t row_sum_up_to(int32_t v)
{
    v += lanes_below<0x111, 0xf>(v);
    v += lanes_below<0x112, 0xf>(v);
    v += lanes_below<0x114, 0xf>(v);
    v += lanes_below<0x118, 0xf>(v);
    return v;
}
// Sum of the threads before this one; *total: of all.  One barrier; `sums` is used once a launch.
__device__ __forceinline__ int32_t sum_before(int32_t *sums, int32_t own, int32_t *total)
{
    const int32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    int32_t up_to = row_sum_up_to(own);
    up_to += lanes_below<0x142, 0xa>(up_to);
    up_to += lanes_below<0x143, 0xc>(up_to);
    if (lane == 63) sums[wave] = up_to;
    lds_barrier();
    const int32_t k = lane & 15, of_wave = k < waves ? sums[k] : 0;
    *total = __builtin_amdgcn_readlane(row_sum_up_to(of_wave), 15);
    return up_to - own + __builtin_amdgcn_readlane(row_sum_up_to(k < wave ? of_wave : 0), 15);
}

struct OrderGeom {
    int32_t N, M, n_index;
    int32_t n_keys, sub_bits;     // buckets: n_keys << sub_bits, by key and the upper sub_bits of the order key
    int32_t top;                  // weight of a key's last chunk index (0: keys have none)
};

// KEYED: chunk-index round: groups of at most M participants with the same key, which gets the peer's position
// in its group as its last chunk index (keys: base-M numbers, first index lowest); *n_groups of them.  Otherwise the permutation:
// index[rank] = peer, -1 where the mask leaves the peer out.  PER: peers of a thread.
template <bool KEYED, int PER>
__global__ __launch_bounds__(kThreads) void small_order_kernel(OrderGeom g, uint64_t seed, int64_t t, int32_t masked,
                                                               typename std::conditional<PER == 1, FewPeerBits, PeerBits>::type bits,
                                                               int32_t *__restrict__ keys, int32_t *__restrict__ index,
                                                               int32_t *__restrict__ n_groups)
{
    extern __shared__ __align__(16) char lds[];
    auto &sh = *reinterpret_cast<Shared<PER * kThreads> *>(lds);
    const int32_t tid = threadIdx.x, lane = tid & 63, T = blockDim.x;
    const int32_t first_of_wave = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int32_t buckets = g.n_keys << g.sub_bits, N = g.N;

    int32_t key[PER];                                        // of the chunk indices
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int32_t i = tid + u * T;
        key[u] = KEYED ? keys[i < N ? i : 0] : 0;
    }
    for (int32_t k = tid; k < buckets; k += T) sh.count[k] = 0;
    if constexpr (KEYED)
        for (int32_t k = tid; k < g.n_index; k += T) sh.list[k] = kNobody;
    if (tid == 0) sh.crowded = 0;
    lds_barrier();

    const uint64_t round_key = mix64(seed + 0xD1B54A32D192ED03ull * static_cast<uint64_t>(t + 1));
    int32_t bucket[PER], at[PER];                            // bucket < 0: the peer is not ranked
    uint64_t order[PER];
    bool present[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        // (64 peers to a wave: two words of the argument block through the scalar cache)
        const int32_t i = tid + u * T, first = first_of_wave + u * T;
        const uint64_t word = first < N ? bits.word[first >> 5] | static_cast<uint64_t>(bits.word[(first >> 5) + 1]) << 32 : 0;
        present[u] = i < N && (masked == 0 || ((word >> lane) & 1u) != 0);
        order[u] = mix64(round_key ^ static_cast<uint64_t>(i));
        const uint32_t sub = g.sub_bits == 0 ? 0u : static_cast<uint32_t>(order[u] >> (64 - g.sub_bits));
        bucket[u] = i < N && (!KEYED || present[u]) ? static_cast<int32_t>(static_cast<uint32_t>(key[u]) << g.sub_bits | sub) : -1;
        at[u] = bucket[u] >= 0 ? atomicAdd(&sh.count[bucket[u]], 1) : 0;
    }
    lds_barrier();

    // first positions of the buckets; four to a thread
    {
        int32_t c[4], sum = 0, total;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = tid * 4 + u;
            c[u] = k < buckets ? sh.count[k] : 0;
            if (c[u] > kCrowded) sh.crowded = 1;
            sum += c[u];
        }
        int32_t before = sum_before(sh.wave_sums[0], sum, &total);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = tid * 4 + u;
            if (k < buckets) sh.start[k] = before;
            before += c[u];
        }
        if (tid == 0) sh.start[buckets] = total;
    }
    lds_barrier();
    const bool crowded = __builtin_amdgcn_readfirstlane(sh.crowded) != 0;        // the same for the whole block

    int32_t begin[PER], n[PER];                              // the peers it is ranked among
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int32_t b = bucket[u] >= 0 ? bucket[u] : 0;
        begin[u] = sh.start[b];
        n[u] = sh.start[b + 1] - begin[u];
    }
    if (crowded) {
        for (int32_t k = tid; k <= N; k += T) sh.slot[k] = 0;
        lds_barrier();
        int32_t slot[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            // (next 32 bits) / 2^32 of the way through the bucket, rounded down: ascending with the order key
            slot[u] = begin[u] + static_cast<int32_t>(__umulhi(static_cast<uint32_t>((order[u] << g.sub_bits) >> 32), static_cast<uint32_t>(n[u])));
            if (bucket[u] >= 0) at[u] = atomicAdd(&sh.slot[slot[u]], 1);
        }
        lds_barrier();
        int32_t c[4], sum = 0, total;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = tid * 4 + u < N ? sh.slot[tid * 4 + u] : 0;
            sum += c[u];
        }
        int32_t before = sum_before(sh.wave_sums[2], sum, &total);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (tid * 4 + u <= N) sh.slot[tid * 4 + u] = before;
            before += c[u];
        }
        if (tid == 0) sh.slot[N] = total;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int32_t s = bucket[u] >= 0 ? slot[u] : 0;
            begin[u] = sh.slot[s];
            n[u] = sh.slot[s + 1] - begin[u];
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (bucket[u] >= 0) sh.order[begin[u] + at[u]] = order[u];
    // first groups of the keys; a key with c members has ceil(c / M)
    if constexpr (KEYED) {
        int32_t c[4], sum = 0, total;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = tid * 4 + u;
            c[u] = k < g.n_keys ? (sh.start[(k + 1) << g.sub_bits] - sh.start[k << g.sub_bits] + g.M - 1) / g.M : 0;
            sum += c[u];
        }
        int32_t before = sum_before(sh.wave_sums[1], sum, &total);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = tid * 4 + u;
            if (k < g.n_keys) sh.group[k] = before;
            before += c[u];
        }
        if (tid == 0) *n_groups = total;
    }
    lds_barrier();

#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (bucket[u] < 0) continue;
        const int32_t i = tid + u * T;
        int32_t rank = begin[u];
        for (int32_t k = begin[u]; k < begin[u] + n[u]; ++k) rank += sh.order[k] < order[u] ? 1 : 0;
        if constexpr (KEYED) {
            rank -= sh.start[key[u] << g.sub_bits];                  // among the peers with its key
            const int32_t chunk = rank % g.M;                        // c_i: position within its group of at most M
            sh.list[(sh.group[key[u]] + rank / g.M) * g.M + chunk] = static_cast<uint16_t>(i);
            keys[i] = key[u] / g.M + chunk * g.top;
        } else {
            sh.list[rank] = static_cast<uint16_t>(present[u] ? i : kNobody);
        }
    }
    lds_barrier();
    for (int32_t k = tid; k < g.n_index; k += T) index[k] = sh.list[k] == kNobody ? -1 : sh.list[k];
}

// log2 of the buckets a key is divided into: about a peer to a bucket
int32_t sub_buckets(int64_t N, int64_t n_keys)
{
    int64_t most = 64;
    while (most < N) most *= 2;
    int32_t b = 0;
    while ((n_keys << (b + 1)) <= most) ++b;
    return b;
}

template <bool KEYED, int PER>
hipError_t launch(const OrderGeom &g, uint64_t seed, int64_t t, const PeerBits *bits, int32_t *keys, int32_t *index, int32_t *n_groups,
                  hipStream_t stream)
{
    const auto kernel = small_order_kernel<KEYED, PER>;
    constexpr int kLds = sizeof(Shared<PER * kThreads>);
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernel), kLds);
    if (e != hipSuccess) return e;
    const int32_t threads = g.N < kThreads ? (g.N + 63) / 64 * 64 : kThreads;
    typename std::conditional<PER == 1, FewPeerBits, PeerBits>::type mask{};
    if constexpr (PER == 1) {
        if (bits != nullptr) mask = few_bits(*bits);
    } else {
        if (bits != nullptr) mask = *bits;
    }
    kernel<<<dim3(1), dim3(threads), kLds, stream>>>(g, seed, t, bits != nullptr, mask, keys, index, n_groups);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_small_permutation(uint64_t seed, int64_t t, int64_t N, const PeerBits *bits, int32_t *perm,
                                    hipStream_t stream)
{
    if (N <= 0 || N > kSmallOrderPeers) return hipErrorInvalidValue;
    const OrderGeom g{static_cast<int32_t>(N), 1, static_cast<int32_t>(N), 1, sub_buckets(N, 1), 0};
    return N <= kThreads ? launch<false, 1>(g, seed, t, bits, nullptr, perm, nullptr, stream)
                         : launch<false, 4>(g, seed, t, bits, nullptr, perm, nullptr, stream);
}

hipError_t launch_small_grouping(int64_t N, int32_t M, int32_t d, uint64_t seed, int64_t t, const PeerBits *bits,
                                 int32_t *keys, int32_t *index, int64_t n_index, int32_t *n_groups, hipStream_t stream)
{
    int64_t n_keys = 1, top = d > 1 ? 1 : 0;
    for (int32_t q = 0; q + 1 < d; ++q) n_keys *= M;
    for (int32_t q = 0; q + 2 < d; ++q) top *= M;
    if (N <= 0 || N > kSmallOrderPeers || n_keys * M != N || n_index != (N / M + n_keys) * M) return hipErrorInvalidValue;
    const OrderGeom g{static_cast<int32_t>(N), M, static_cast<int32_t>(n_index), static_cast<int32_t>(n_keys), sub_buckets(N, n_keys),
                      static_cast<int32_t>(top)};
    return N <= kThreads ? launch<true, 1>(g, seed, t, bits, keys, index, n_groups, stream)
                         : launch<true, 4>(g, seed, t, bits, keys, index, n_groups, stream);
}

}  // namespace moshpit
