// Tiles of the distortion's pass over a state (dist_to_mean.hip): host arithmetic on plain numbers, without GPU types.
#pragma once

#include <stdint.h>

namespace moshpit {

struct DistTiles {
    int32_t lanes, waves;        // 16-byte vectors of a row in a tile; waves of a block, which share its rows
    int64_t blocks;
    bool streaming;              // non-temporal loads
    bool last_first;             // rows are taken from the last to the first
};

// Tiles for N rows of P elements; whole_lines: rows start on cache lines.  false: rows of less than a vector, or too many of
// them for 32-bit row numbers.  From sweeps on MI355X (8 to 64 lanes, 1 to 8 waves, both kinds of loads; 9 to 4096 rows, 0.4 MB
// to 1.6 GB, on and off the cache lines), us:
//   Tiles as wide as leaves 160 of them (130 of large states), whose 8 waves a block then make 1,300 on the chip: 4096 rows, 400 MB, 32 lanes x 8
//   waves 60, 8 x 1 64; 1024 rows, 25 MB, 8 x 8 8.2, 16 x 8 9.6; 512 rows, 100 MB, 64 x 8 18.0, 16 x 1 19.1.  A block of several
//   waves ends with barriers for every element of a vector, so bfloat16 states of up to 256 rows and 40 MB take one wave, whose
//   lanes share more rows the more there are: 32 rows, 1.6 MB, 32 x 1 7.9, 8 x 4 10.7; 64 rows, 25 MB, 32 x 1 9.4, 8 x 4 27; 144
//   rows, 1.6 MB, 16 x 1 8.8, 32 x 1 10.7, 8 x 8 9.9; 256 rows, 6.4 MB, 8 x 1 8.8, 16 x 1 10.5, 8 x 8 10.1.
//   Waves until the chip has 1,000: 256 rows, 400 MB, 1 wave 64.5, 8 waves 73.5; 1024 rows, 25 MB binary32, 8 waves 8.2, 4
//   waves 8.8.  From 550 MB on 64 lanes and waves until the chip has 1,100: the last-level cache is full of what wrote the state, and
//   the lines that a pass pushes out of it cost most with more than 2,050 waves in flight (the pass that follows the write : the next
//   one; 4096 rows of 2.1 GB bfloat16 1,002 waves 387 : 395, 2,004 313 : 308, 4,008 340 : 316; 576 rows of 2.1 GB binary32 64 x 8 423 :
//   311, 64 x 1 340 : 313; 1024 rows of 4.2 GB bfloat16 64 x 8 748 : 616, 64 x 1 644 : 621).  Where that would be two waves, whole
//   lines of bfloat16 take tiles of half the width (2048 rows of 1.4 GB 64 x 2 270 : 214, 32 x 1 219 : 216; 4096 rows of 3 GB 549 : 452 and 460 : 453).
//   Beyond 1 GB under 128 rows of binary32 8 waves, if a wave then still has a load of 8 rows (64 rows, 2.1 GB, 1 wave 404 : 311, 8 waves 383 : 306).
//   Fewer than 32 rows are a load or two of a wide tile: 16 rows, 6.4 MB bfloat16, 32 x 1 6.9, 8 x 4 9.4.
//   Never more than 65,536 tiles where they can be wider (their sums take one block 10 us).
//   Non-temporal loads beyond 64 MB (4096 rows, 1.6 GB 231 : 250; 1024 rows, 25 MB 9.4 : 8.2), but where neighbours share cache lines
//   only in 1 KiB tiles of 32 rows and more (1024 rows, 1.6 GB, 32 lanes 281 : 262, 64 lanes 248 : 258; 144 rows 256 : 269; 9 rows, 100 MB
//   22.5 : 20.8), which such states take as soon as there are enough.  From 350 MB on the last-level cache no longer helps rows off
//   the lines either: 64 lanes and non-temporal loads, of 1024 rows (bfloat16 512) and more 32 lanes where there are 500 such tiles (the pass that
//   follows the write : the next one, ordinary loads of 32 lanes against that: 256 rows, 450 MB bfloat16 96 : 84, 78 : 77, 370 MB 79 : 70, 65 : 64;
//   2048 rows, 540 MB binary32 133 : 104, 116 : 102, in 64 lanes 126 : 116).
//   Rows from the first to the last, but the other way round from 270 to 700 MB, of whose last rows the last-level cache holds many, and binary32 of
//   700 rows, bfloat16 of 2048 rows and more (the pass that follows the write, first to last : last to first; 256 rows, 1 GB 189 : 194, 64 to
//   576 rows of 0.7 to 4 GB 1 to 3 % on average; 576 rows, 360 MB binary32 63 : 59, 256 rows, 370 MB bfloat16 off the lines 79 : 75; 2048 rows
//   of binary32 2 to 3 %, 4096 rows of 2.1 GB bfloat16 371 : 359, but 4 GB 657 : 683; the next pass within 1 % either way).
inline bool dist_tiles(int64_t esize, int64_t N, int64_t P, bool whole_lines, DistTiles *out)
{
    const int64_t row = P * esize;
    if (row < 16 || N > (int64_t(1) << 30)) return false;
    const int64_t vectors = (row + 15) / 16;
    const double state = static_cast<double>(N) * static_cast<double>(row);
    const bool f32 = esize == 4, few = N < 32, large = !few && state > 5.5e8, odd_lines = !few && !whole_lines && state > 3.5e8;
    int32_t lanes = few ? (f32 || N <= 12 ? 64 : 32) : f32 && N < 1024 ? 64 : 32;
    if (large || (!whole_lines && !few && f32 && vectors >= 65536)) lanes = 64;
    if (large && !f32 && whole_lines && vectors > 64 * 550 && vectors <= 64 * 1000) lanes = 32;
    if (odd_lines && !large) lanes = N >= (f32 ? 1024 : 512) && vectors >= 500 * 32 ? 32 : 64;
    const bool one_wave = !f32 && !few && N <= 256 && state < 40e6;
    if (one_wave) lanes = N <= 64 ? 32 : N <= 160 ? 16 : 8;
    const int64_t least = large ? 130 : f32 || N >= 512 ? 160 : 512;
    while (!few && !one_wave && lanes > 8 && vectors < least * lanes) lanes /= 2;
    while (lanes < 64 && vectors > 65536ll * lanes) lanes *= 2;
    const int64_t blocks = (vectors + lanes - 1) / lanes;
    if (blocks > 0x7fffffffll) return false;
    int32_t waves = 1;
    const auto twice = [&] { return waves < 8 && N >= 2 * waves * (64 / lanes); };           // (a row for every lane)
    while (!few && !one_wave && twice() && (blocks * waves < (large ? 1100 : 1000) || (state > 1e9 && f32 && N >= 64 && N < 128))) waves *= 2;
    out->lanes = lanes;
    out->waves = waves;
    out->blocks = blocks;
    out->streaming = state > 64e6 && (whole_lines || (lanes == 64 && !few) || odd_lines);
    out->last_first = N >= (f32 ? 700 : 2048) || (state > 2.7e8 && state < 7e8);
    return true;
}

}  // namespace moshpit
