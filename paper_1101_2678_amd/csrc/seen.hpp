// seen.hpp -- the visited set as byte flags in LDS, for the kernels whose usual
// step reads a short list, and the bits that their step on a whole row makes
// from them.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace aco {
namespace {

// Visited flags: one byte a city of the row's passes, 1 = visited or beyond
// n.  A visit is one byte store, and a listed city's flag one byte load at
// the city itself.
__host__ __device__ size_t seen_lds_bytes(int n) { return ((size_t)n + 511) & ~(size_t)511; }

// Visited flags of the ant's first `cities` cities (a multiple of 512): 0, or
// 1 beyond n.
__device__ __forceinline__ uint8_t* clear_flags(uint8_t* s_seen, int n, int cities, int lane) {
    for (int w = lane; w < cities / 4; w += 64) {
        uint32_t f = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) f |= (4 * w + e >= n ? 1u : 0u) << (8 * e);
        reinterpret_cast<uint32_t*>(s_seen)[w] = f;
    }
    __builtin_amdgcn_wave_barrier();
    return s_seen;
}

// The lane and block bits of the general step from the flags of the ant's P
// passes.  s_bits: 64 P bytes of scratch.
template <int P, typename B>
__device__ __forceinline__ void bits_from_flags(const uint2* s_seen, uint8_t* s_bits, int lane,
                                                B& lane_bits, uint64_t& block_bits) {
    // four bytes of 0 or 1 to four bits
    const auto four = [](uint32_t x) { return (x * 0x10204080u) >> 28; };
    uint32_t seen[P];
    lane_bits = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint2 f = s_seen[64 * p + lane];  // cities 512 p + 8 lane .. + 7
        seen[p] = four(f.x) | four(f.y) << 4;
        lane_bits |= (B)(seen[p] ^ 0xFFu) << (8 * p);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) s_bits[64 * p + lane] = (uint8_t)seen[p];
    // block b: the eight bytes from 8 b
    block_bits = ~0ull;
    if (lane < 8 * P) {
        block_bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) block_bits |= (uint64_t)s_bits[8 * lane + e] << (8 * e);
    }
}

}  // namespace
}  // namespace aco
