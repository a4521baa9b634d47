// construct_flat.hpp -- the roulette step for short rows: one city of every
// 64-city block per lane.
//
// Lane l holds city 64 b + l of each of the row's B blocks, so a block's S64
// prefixes are one scan in place, the visited set is B scalar words used
// directly as lane masks, and nothing goes through LDS or between lanes but
// the scans (the tiled layout of longer rows sums blocks across lanes first
// and then rescans the chosen one).  All B blocks are scanned, side by side,
// so the chain of a step is that of one scan as long as B is small.
#pragma once

#include "r64_lanes.hpp"

namespace aco {
namespace {

// Rows of up to 64 times this many cities.  One construction with m = n,
// tiled / flat: n = 64 0.0261 / 0.0180 ms, n = 100 0.0391 / 0.0276, n = 128
// 0.0484 / 0.0335, n = 192 0.0710 / 0.0548, n = 256 0.0927 / 0.0817, n = 320
// 0.137 / 0.123; n = 384 0.155 / 0.169 (every block costs six adds more).  With
// the factors (construct_masked.hpp) n = 320 takes 0.119, so the fifth block is
// for tile 4 and the batched launch, which has none.
constexpr int kMaxFlatBlocks = 5;

// x of the lanes whose bit of `mask` (wave-uniform) is set, else +0.
__device__ __forceinline__ float keep_lanes(float x, uint64_t mask) {
    float y;
    asm("v_cndmask_b32 %0, 0, %1, %2" : "=v"(y) : "v"(x), "s"(mask));
    return y;
}

// The lowest set bit of `mask`, or ~0 if there is none (the instruction's own
// result).
__device__ __forceinline__ uint32_t first_lane(uint64_t mask) {
    uint32_t r;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(mask));
    return r;
}

// The unvisited cities of an ant on a row of B blocks: bit t of word b is
// city 64 b + t.  Wave-uniform.
template <int B>
struct Unvisited {
    uint64_t word[B];
    __device__ __forceinline__ explicit Unvisited(int n) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int valid = n - 64 * b;
            word[b] = valid >= 64 ? ~0ull : valid <= 0 ? 0ull : (1ull << valid) - 1ull;
        }
    }
    // a lane compare and a scalar AND a word
    __device__ __forceinline__ void visit(int city, int lane) {
#pragma unroll
        for (int b = 0; b < B; ++b) word[b] &= ballot(64 * b + lane != city);
    }
    // from one byte a city, 0 = unvisited
    __device__ __forceinline__ void from_flags(const uint8_t* seen, int lane) {
        bool live[B];
#pragma unroll
        for (int b = 0; b < B; ++b) live[b] = seen[64 * b + lane] == 0;
#pragma unroll
        for (int b = 0; b < B; ++b) word[b] = ballot(live[b]);
    }
};

// The row's loads: the padding past n reads as zeros or, past the span, as
// nothing, and the masks drop it either way.  (A copy of the matrix in LDS for
// four ants at a time was 15% faster to n = 64 and 6 to 20% slower from there
// to n = 200.)
template <int B>
__device__ __forceinline__ void load_flat(const float* __restrict__ mat, int records, int row,
                                          int row_bytes, int lane, uint32_t (&x)[B]) {
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(mat, records);
    const int soff = row * row_bytes;
#pragma unroll
    for (int b = 0; b < B; ++b)
        x[b] = __builtin_amdgcn_raw_buffer_load_b32(rs, (64 * b + lane) * 4, soff, 0);
}

// One R64 draw over a loaded row.  Returns the chosen city, or -1 if none is
// unvisited.  Wave-uniform.
template <int B>
__device__ __forceinline__ int pick_flat(const uint32_t (&x)[B], const Unvisited<B>& live,
                                         float u) {
    float s[B], t[B];
#pragma unroll
    for (int b = 0; b < B; ++b) s[b] = keep_lanes(__uint_as_float(x[b]), live.word[b]);
    s64_scans<B>(s);
    // S64 over the block totals, which lane 63 holds: a Kogge-Stone scan
#pragma unroll
    for (int b = 0; b < B; ++b) t[b] = s[b];
#pragma unroll
    for (int d = 1; d < B; d <<= 1)
#pragma unroll
        for (int b = B - 1; b >= d; --b) t[b] = t[b] + t[b - d];
    // opaque, or the product becomes a scalar read, a move and a product
    float goal = u * t[B - 1];
    asm("" : "+v"(goal));
    const float target = read_lane(goal, 63);
    // the lowest city with a hit: first_lane is ~0 for a block without one
    uint32_t j = first_lane(ballot(s[0] > target) & live.word[0]);
#pragma unroll
    for (int b = 1; b < B; ++b) {
        const uint32_t h =
            first_lane(ballot(read_lane(t[b - 1], 63) + s[b] > target) & live.word[b]) | 64 * b;
        j = h < j ? h : j;
    }
    if (__builtin_expect((int)j < 0, 0)) {
        // no prefix exceeds the target: the highest unvisited city, or -1
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (live.word[b]) j = 64 * b + 63 - __builtin_clzll(live.word[b]);
    }
    return (int)j;
}

}  // namespace
}  // namespace aco
