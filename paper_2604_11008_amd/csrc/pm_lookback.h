// pm_lookback.h -- index arithmetic of the look-back over a segment's tiles
// (library-internal; plain integer functions, so that a host program can run
// them too).
//
// A walk from tile q of a segment whose first tile is q0 adds up the leavers of
// the tiles before q, in rounds from `end` (at first q) downwards.  In a round
// every lane of a wave reads what one block of 64 tiles handed on (the
// segment's leavers up to the block's end, + 1, or 0: not yet) and kWalkWords
// words of four tiles' statuses each (a tile's leavers + 1 in 16 bits, or 0).
// The k-th lane's block is the k-th before `end`, so the lowest lane whose block
// has handed on says where the adding up ends.
#ifndef PM_LOOKBACK_H
#define PM_LOOKBACK_H

#include <stdint.h>

namespace pm {

constexpr int kWalkWords = 4;

// The lane's block, counted from the segment's first; -1 stands for the
// segment's start (nothing before it), lower ones for nothing.
__host__ __device__ __forceinline__ int walk_block(int q0, int end, int lane)
{
    return ((end - q0) >> 6) - 1 - lane;
}

// The lane's i-th word: tiles 4 w to 4 w + 3.  Only those with a tile of the
// segment are read.
__host__ __device__ __forceinline__ int walk_word(int end, int lane, int i)
{
    return ((end + 3) >> 2) - 1 - lane - 64 * i;
}

__host__ __device__ __forceinline__ bool walk_reads(int q0, int w) { return 4 * w + 4 > q0; }

// The first tile to add up where the k-th lane's block is the nearest that has
// handed on (k = 63 where none has: that block's end is as far as it goes).
__host__ __device__ __forceinline__ int walk_from(int q0, int end, int k)
{
    const int start = q0 + (((end - q0) >> 6) - k) * 64;
    return start > q0 ? start : q0;
}

// The first tile that the words of a round hold.
__host__ __device__ __forceinline__ int walk_low(int end)
{
    return 4 * ((end + 3) >> 2) - 256 * kWalkWords;
}

// The fields of word w that belong to tiles [from, end).
__host__ __device__ __forceinline__ uint64_t walk_mask(int w, int from, int end)
{
    const int lo = from - 4 * w, hi = end - 4 * w;
    const int f0 = lo < 0 ? 0 : (lo > 4 ? 4 : lo);
    const int f1 = hi < 0 ? 0 : (hi > 4 ? 4 : hi);
    return f0 < f1 ? (~0ull >> (64 - 16 * (f1 - f0))) << (16 * f0) : 0ull;
}

// Whether one of the masked fields of a word is not yet known.
__host__ __device__ __forceinline__ bool walk_missing(uint64_t word, uint64_t mask)
{
    const uint64_t x = word | ~mask;
    return ((x - 0x1000100010001ull) & ~x & 0x8000800080008000ull) != 0;
}

// The leavers of the masked fields, all known.
__host__ __device__ __forceinline__ uint32_t walk_sum(uint64_t word, uint64_t mask)
{
    // less 1 for each field (a field is at least 1 where the mask is set)
    uint64_t x = (word & mask) - (mask & 0x1000100010001ull);
    x = (x & 0xffff0000ffffull) + ((x >> 16) & 0xffff0000ffffull);
    return (uint32_t)x + (uint32_t)(x >> 32);
}

}  // namespace pm

#endif  // PM_LOOKBACK_H
