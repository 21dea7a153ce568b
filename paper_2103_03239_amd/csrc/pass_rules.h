// Sizes and choices of multi-round passes: host arithmetic on plain numbers, without GPU types.
#pragma once

#include <stdint.h>

namespace moshpit {

// Tables of whole-grid passes (who takes part in which round, who copies whom) are built for a
// bounded number of rounds at a time, so that their memory and the launch that fills them do not
// grow with the length of a run: 16 MiB hold 16,000 rounds of 16 x 16 x 16 peers, 900 with refresh.
constexpr int64_t kGridTableBytes = int64_t(16) << 20;
constexpr int64_t kGridTableRounds = 65536;            // (the launch has one block per round)

// Per round: a 32-bit bitmap per group; with refresh a list of at most N pairs and its length.
inline int64_t grid_table_round_bytes(int64_t N, int32_t M, bool refresh)
{
    return 4 * (N / M) + (refresh ? 4 * N + 4 : 0);
}

// Rounds the tables are built for at once: whole passes of max_rounds rounds, at least one.
inline int64_t grid_table_rounds(int64_t N, int32_t M, bool refresh, int64_t max_rounds)
{
    int64_t n = kGridTableBytes / grid_table_round_bytes(N, M, refresh);
    if (n > kGridTableRounds) n = kGridTableRounds;
    n = n / max_rounds * max_rounds;
    return n < max_rounds ? max_rounds : n;
}

// A pass leaves one partial sum per tile for every distortion it computes; they are summed before
// the next pass, so the buffer holds those of one pass, and a pass over a state so wide that they
// would take more than 256 MiB takes fewer rounds.
constexpr int64_t kGridPartialBytes = int64_t(256) << 20;

inline int32_t grid_pass_rounds(int32_t max_rounds, int64_t entry_tiles)
{
    if (entry_tiles <= 0) return max_rounds;
    const int64_t n = kGridPartialBytes / (8 * entry_tiles) - 1;
    return n < 1 ? 1 : n < max_rounds ? static_cast<int32_t>(n) : max_rounds;
}

}  // namespace moshpit
