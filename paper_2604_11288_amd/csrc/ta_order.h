// Order in which workgroups take the units of a launch.
#pragma once
#include "ta_internal.h"

namespace ta {

// Division of numbers below 2^31 by one that the host knows: a multiplication and a shift in the scalar unit, where the
// compiler's own takes some forty dependent vector instructions (four of those were half a microsecond of every workgroup).
// mul = ceil(2^(31 + l) / d) with 2^l >= d is too large by less than one part in 2^31, so the quotient is exact.
struct Divider {
    uint32_t mul, shift;
};

inline Divider divider(uint32_t d)
{
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}

__device__ __forceinline__ uint32_t divide(uint32_t x, const Divider& by) { return (uint32_t)(((uint64_t)x * by.mul) >> by.shift); }

// A launch's dimension holds fewer than 2^32 threads, 2^24 workgroups of 256: a longer row of workgroups goes in lines of GRID_LINE, the last
// of them padded.
constexpr uint32_t GRID_LINE = 1u << 23;
struct GridLines {
    uint32_t x, lines;
    explicit GridLines(int64_t blocks)
        : x(blocks < (int64_t)GRID_LINE ? (uint32_t)blocks : GRID_LINE), lines((uint32_t)((blocks + GRID_LINE - 1) / GRID_LINE)) {}
};

// The unit that comes `at`-th: as numbered when all sequences are equally long, else all units of the longest sequence
// first, then those of the next (equal lengths in batch order).  The longest units then start first and the shortest fill the
// gaps at the end, and a compute unit's second workgroup is shorter than its first.  Every wavefront works the order out for
// itself from the lengths, one lane per sequence (so up to 64 sequences; more stay in their own order).
__device__ __forceinline__ int32_t unit_at(int32_t at, const int32_t* seq_len, int32_t batch, int32_t hkv, int32_t units)
{
    if (!seq_len || batch < 2 || batch > 64) return at;
    const int32_t per_seq = units / batch;                     // layers * hkv
    const int32_t rank = at / per_seq, pair = at - rank * per_seq;
    const int lane = (int)(threadIdx.x & 63u);
    const int32_t len = lane < batch ? seq_len[lane] : 0;
    int32_t longer = 0;                                        // sequences that come before this lane's
    for (int j = 0; j < batch; ++j) {
        const int32_t other = __builtin_amdgcn_readlane(len, j);
        longer += other > len || (other == len && j < lane) ? 1 : 0;
    }
    const unsigned long long hit = __ballot(lane < batch && longer == rank);
    const int32_t b = (int32_t)__ffsll((long long)hit) - 1;
    const int32_t l = pair / hkv, g = pair - l * hkv;
    return (l * batch + b) * hkv + g;
}

// Workgroup -> place in that order: block b runs on XCD b mod 8, and the `parts` workgroups of a unit on one XCD.
__device__ __forceinline__ int32_t place_of(uint32_t block, int32_t parts, const Divider& by_parts, int32_t& part)
{
    const int32_t in_xcd = (int32_t)(block >> 3);
    const int32_t k = (int32_t)divide((uint32_t)in_xcd, by_parts);
    part = in_xcd - k * parts;
    return k * 8 + (int32_t)(block & 7u);
}

}  // namespace ta
