// construct_masked.hpp -- the roulette step for rows of one to three passes of
// 512 cities: the tiled layout with the visited set as factors in LDS, for
// launches whose ants fit the device in one round (masked_rows).
//
// The step of such a row is bound by the instructions of its one wavefront,
// and half of them made masks: two for every city.  Here the ant keeps a
// factor a city in LDS, 1 or +0; a lane reads those of its cities with the
// row's own loads still in flight, and they enter the block sums as
// multiplications (exact: w * 1 = w, w * +0 = +0), one fused with the pair's
// addition: fl(w0 f0 + w1 f1) with both products exact is fl(w0 + w1) of the
// masked weights, so every block total has the same bits.  A visit is one
// store.  Bits / factors, m = n, first iteration (whole rows): n = 400
// 0.171 -> 0.149 ms, n = 700 0.356 -> 0.325, n = 1000 0.516 -> 0.485, n =
// 1500 1.37 -> 1.28.
#pragma once

#include "construct_flat.hpp"
#include "r64_lanes.hpp"

namespace aco {
namespace {

constexpr int kMaxMaskedPasses = 3;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Factors of the cities of P passes: 1, or 0 beyond n.
template <int P>
__device__ __forceinline__ void init_factors(float* s_f, int n, int lane) {
#pragma unroll
    for (int p = 0; p < 8 * P; ++p) s_f[64 * p + lane] = 64 * p + lane < n ? 1.0f : 0.0f;
    __builtin_amdgcn_wave_barrier();
}

// fl32 sums of masked weights, as pair_sum4 of the masked vector.
__device__ __forceinline__ float masked_sum4(const u32x4& w, const f32x4& f) {
    const float a = __builtin_fmaf(__uint_as_float(w.y), f.y, __uint_as_float(w.x) * f.x);
    const float b = __builtin_fmaf(__uint_as_float(w.w), f.w, __uint_as_float(w.z) * f.z);
    return a + b;
}

// The row's loads: in pass p lane l takes cities 512 p + 8 l .. + 7.
template <int P>
__device__ __forceinline__ void load_passes(const float* __restrict__ mat, int records, int row,
                                            int row_bytes, int lane, u32x4 (&wa)[P],
                                            u32x4 (&wb)[P]) {
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(mat, records);
    const int soff = row * row_bytes;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        wa[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, (512 * p + 8 * lane) * 4, soff, 0);
        wb[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, (512 * p + 8 * lane) * 4 + 16, soff, 0);
    }
}

// One R64 draw over a loaded row.  s_w: 512 P words, the row as loaded; s_T: 64
// words, 0 past the row's blocks.  Returns the chosen city, or -1 if none is
// unvisited.  Wave-uniform.
template <int P>
__device__ __forceinline__ int pick_masked(const u32x4 (&wa)[P], const u32x4 (&wb)[P], int n,
                                           const float* s_f, float* s_T, float* s_w, float u,
                                           int lane) {
    f32x4 fa[P], fb[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const f32x4* f = reinterpret_cast<const f32x4*>(s_f + 512 * p + 8 * lane);
        fa[p] = f[0];
        fb[p] = f[1];
    }
    const int nb = (n + 63) >> 6;
    float t[P];
#pragma unroll
    for (int p = 0; p < P; ++p) t[p] = masked_sum4(wa[p], fa[p]) + masked_sum4(wb[p], fb[p]);
#pragma unroll
    for (int p = 0; p < P; ++p) t[p] = group_pairwise<8>(t[p]);
    // block b = 8 p + g, the total in lane 8 g + 7, to lane b
    float T = 0.0f;
    if constexpr (P == 1) {
        if ((lane & 7) == 7) s_T[lane >> 3] = t[0];
        T = s_T[lane];
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float x = __int_as_float(
                __builtin_amdgcn_ds_bpermute(((lane & 7) * 8 + 7) * 4, __float_as_int(t[p])));
            T = lane >> 3 == p ? x : T;
        }
        __builtin_amdgcn_sched_barrier(0x7F);  // no LDS store above those reads
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        u32x4* dst = reinterpret_cast<u32x4*>(s_w + 512 * p + 8 * lane);
        dst[0] = wa[p];
        dst[1] = wb[p];
    }
    float I;
    if constexpr (P <= 2)
        I = s64_scan_row0_levels<block_scan_levels(8 * P)>(T);
    else
        I = s64_scan(T);
    // opaque, or the product becomes a scalar read, a move and a product
    float goal = u * I;
    asm("" : "+v"(goal));
    const float target = read_lane(goal, nb - 1);
    const float E = wave_shift_up1(I);
    uint64_t cand = ballot(E + T * kBlockSlack > target) & ((1ull << nb) - 1ull);
    // the chosen city if block b holds it, else a negative number
    const auto in_block = [&](int b) {
        const float f = s_f[64 * b + lane];
        const float s = s64_scan(s_w[64 * b + lane] * f);
        const uint64_t hit = ballot(read_lane(E, b) + s > target) & ballot(f != 0.0f);
        return (int)(first_lane(hit) | (uint32_t)(64 * b));
    };
    // nearly always the first candidate block holds it
    int j = -1;
    if (__builtin_expect(cand != 0, 1)) j = in_block(__builtin_ctzll(cand));
    if (__builtin_expect(j < 0, 0)) {
        for (cand &= cand - 1; cand != 0 && j < 0; cand &= cand - 1)
            j = in_block(__builtin_ctzll(cand));
        // no prefix exceeds the target: the highest unvisited city
        for (int b = nb - 1; b >= 0 && j < 0; --b) {
            const uint64_t live = ballot(s_f[64 * b + lane] != 0.0f);
            if (live) j = 64 * b + 63 - __builtin_clzll(live);
        }
    }
    return j;
}

}  // namespace
}  // namespace aco
