// construct_product.hip -- tour construction with the paper's data-parallel
// selection (Section III-A; Table II, versions 7-8): every unvisited city j of
// the current row draws its own uniform r_j, the product fl32(choice[i][j] *
// r_j) is formed, and the largest product wins (lowest j among equal ones).
// Visited cities are left out of the reduction rather than multiplied by 0,
// and the tile winners compete on the same product, so the tiling of the row
// over lanes cannot change the result.
//
// r_j = (x >> 8) * 2^-24 with x = word (j mod 4) of Philox4x32-10 at counter
// (step, ant, iter, 1 + j / 4), key = seed: one Philox block serves four
// consecutive cities.
//
// One wavefront per ant.  Where the weights of the rows differ enough, a step
// draws for the 63 largest entries of the row first (one Philox block a lane,
// 512 bytes read): a winner above the largest entry of the rest is the winner of
// the whole row, and nearly every step ends there, bound by the latency of that
// chain.  Otherwise the wave reads the whole row; in pass p lane l holds cities
// 512 p + 8 l .. +7 (two 16-byte loads of the choice row, two Philox blocks).
// All loads of such a step are issued before the first Philox block is
// computed, so the row streams while the vector unit generates the draws; it
// does n / 4 Philox blocks and reads 4n bytes, which makes it bound by integer
// multiply throughput rather than by memory.  Each lane keeps only the largest
// product key of each pass (one max per city); a DPP reduction gives the wave's
// largest key, a ballot per pass finds the lowest pass and lane holding it, and
// that lane's lowest position holding it gives the city.
#include <hip/hip_runtime.h>

#include "aco_device.hpp"
#include "aco_state.hpp"
#include "product.hpp"
#include "seen.hpp"
#include "shortlist.hpp"

namespace aco {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kG = 8;              // cities per lane per pass
constexpr int kPass = 64 * kG;     // cities per pass
constexpr int kMaxPasses = kMaxCities / kPass;

__host__ __device__ size_t tour_bytes(int n) {
    return ((size_t)(n + 1) * sizeof(uint16_t) + 15) & ~(size_t)15;
}

// a ^ b ^ k in one v_bitop3_b32 (truth table 0x96); k is wave-uniform.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t k) {
    uint32_t d;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(d) : "v"(a), "v"(b), "s"(k));
    return d;
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11), all four output words.
// The 32 x 32 -> 64-bit products give both halves in one multiply.  With
// only the last counter word varying across lanes, part of rounds 1-3 is
// wave-uniform and the compiler keeps it on the scalar unit; from round 3
// on every value varies per lane and the two XORs of a word fuse into one
// three-input operation.
// NB Philox blocks that differ only in the last counter word, computed round
// by round across the blocks: NB independent multiply chains per round keep
// the vector unit busy although a SIMD holds only two or three ants.
template <int NB>
__device__ __forceinline__ void philox4_many(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1,
                                             uint32_t c2, const uint32_t (&c3)[NB],
                                             u32x4 (&out)[NB]) {
    uint32_t a[NB], b[NB], c[NB], d[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        a[i] = c0;
        b[i] = c1;
        c[i] = c2;
        d[i] = c3[i];
    }
#pragma unroll
    for (int r = 0; r < 10; ++r) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const uint64_t pa = (uint64_t)0xD2511F53u * a[i];
            const uint64_t pb = (uint64_t)0xCD9E8D57u * c[i];
            uint32_t y0, y2;
            if (r >= 3) {
                y0 = xor3((uint32_t)(pb >> 32), b[i], k0);
                y2 = xor3((uint32_t)(pa >> 32), d[i], k1);
            } else {
                y0 = (uint32_t)(pb >> 32) ^ b[i] ^ k0;
                y2 = (uint32_t)(pa >> 32) ^ d[i] ^ k1;
            }
            a[i] = y0;
            b[i] = (uint32_t)pb;
            c[i] = y2;
            d[i] = (uint32_t)pa;
        }
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) out[i] = u32x4{a[i], b[i], c[i], d[i]};
}

__device__ __forceinline__ float unit24(uint32_t x) { return (float)(x >> 8) * 0x1.0p-24f; }

template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, kCtrl, kRowMask, 0xF, false);
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    x = max(x, dpp_u32<0x111, 0xF>(0u, x));
    x = max(x, dpp_u32<0x112, 0xF>(0u, x));
    x = max(x, dpp_u32<0x114, 0xF>(0u, x));
    x = max(x, dpp_u32<0x118, 0xF>(0u, x));
    x = max(x, dpp_u32<0x142, 0xA>(0u, x));
    x = max(x, dpp_u32<0x143, 0xC>(0u, x));
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
    x = min(x, dpp_u32<0x111, 0xF>(~0u, x));
    x = min(x, dpp_u32<0x112, 0xF>(~0u, x));
    x = min(x, dpp_u32<0x114, 0xF>(~0u, x));
    x = min(x, dpp_u32<0x118, 0xF>(~0u, x));
    x = min(x, dpp_u32<0x142, 0xA>(~0u, x));
    x = min(x, dpp_u32<0x143, 0xC>(~0u, x));
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// City e of lane `lane` in pass p; a lane's cities of a pass are whole Philox
// blocks.
__device__ constexpr int city_of(int p, int lane, int e) { return kPass * p + kG * lane + e; }

// Draws of one step from Philox for lane `lane`: block 1 + q + b
// holds cities 4 (q + b) .. + 3 (q = first city / 4).
struct PhiloxDraws {
    uint32_t k0, k1, step, ant, iter;
    template <int P>
    __device__ __forceinline__ void get_all(int lane, float (&r)[P][kG]) const {
        constexpr int B = kG / 4;  // blocks per lane per pass
        uint32_t ctr[B * P];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int b = 0; b < B; ++b)
                ctr[B * p + b] = 1u + (uint32_t)city_of(p, lane, 0) / 4u + (uint32_t)b;
        u32x4 x[B * P];
        philox4_many<B * P>(k0, k1, step, ant, iter, ctr, x);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) r[p][4 * b + e] = unit24(x[B * p + b][e]);
    }
};

// Draws given in memory (verification entry point): n floats per row.
struct ArrayDraws {
    const float* u;
    int n;
    template <int P>
    __device__ __forceinline__ void get_all(int lane, float (&r)[P][kG]) const {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int e = 0; e < kG; ++e) {
                const int j = city_of(p, lane, e);
                r[p][e] = j < n ? u[j] : 0.0f;
            }
    }
};

// All ones if bit e of `bits` is set, else 0 (one v_bfe_i32).  Inline
// assembly here: through the builtin the compiler scheduled this kernel 3.5%
// slower (n = 2400), while the roulette kernels gained from it.
__device__ __forceinline__ uint32_t bit_mask(uint32_t bits, int e) {
    uint32_t m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(bits), "i"(e));
    return m;
}

// One selection over a whole row: bit kG p + e of `bits` says whether the
// lane's city e of pass p may be chosen.  Products of finite non-negative
// values are finite and non-negative, so their bit patterns order like the
// values; a city that may not be chosen gets key 0.  Returns the wave's
// largest key and the lowest city holding it; if no product of a city that
// may be chosen is positive, key 0 and the lowest city that may be chosen
// (all products equal, so the lowest index wins); city ~0 if there is none.
struct Pick {
    uint32_t key, city;
};

template <int P, typename Draws>
__device__ __forceinline__ Pick product_pick(const float* row, int n, uint64_t bits,
                                             const Draws& draws, int lane) {
    constexpr int L = kG / 4;  // 16-byte loads per lane per pass
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(row), (short)0, ((n + 3) & ~3) * 4, 0x00020000);
    u32x4 wv[P][L];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int b = 0; b < L; ++b)
            wv[p][b] = __builtin_amdgcn_raw_buffer_load_b128(
                rs, (city_of(p, lane, 0) + 4 * b) * 4, 0, 0);
    // every row load above is in flight before the first draw is computed
    __builtin_amdgcn_sched_barrier(0);
    float r[P][kG];
    draws.template get_all<P>(lane, r);
    uint32_t key[P][kG], pmax[P];
    uint32_t lmax = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t pass_bits = (uint32_t)(bits >> (kG * p));
        uint32_t m = 0;
#pragma unroll
        for (int e = 0; e < kG; ++e) {
            const float prod = __uint_as_float(wv[p][e / 4][e % 4]) * r[p][e];
            key[p][e] = __float_as_uint(prod) & bit_mask(pass_bits, e);
            m = max(m, key[p][e]);
        }
        pmax[p] = m;
        lmax = max(lmax, m);
    }
    const uint32_t top = wave_max_u32(lmax);
    if (top != 0u) {
        // cities grow with (pass, lane, position): the first pass with a lane
        // holding top, its lowest such lane, that lane's lowest position
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint64_t hold = ballot(pmax[p] == top);
            if (hold) {
                const int src = __builtin_ctzll(hold);
                uint32_t first = 0;
#pragma unroll
                for (int e = kG - 1; e >= 0; --e) first = key[p][e] == top ? (uint32_t)e : first;
                const int e = __builtin_amdgcn_readlane((int)first, src);
                // wave-uniform; said so, or the next row's address is taken
                // as per-lane and every load of it becomes a loop
                const int city = __builtin_amdgcn_readfirstlane(city_of(p, src, e));
                return Pick{top, (uint32_t)city};
            }
        }
    }
    // No positive product: the lowest city that may be chosen.  Bit kG p + e
    // grows with the city inside a lane.
    uint32_t low = ~0u;
    if (bits) {
        const int b = __builtin_ctzll(bits);
        low = (uint32_t)city_of(b / kG, lane, b % kG);
    }
    return Pick{0u, wave_min_u32(low)};
}

// The selection from the row's short list alone (v: the lane's entry,
// unvisited: whether its city is): the lanes that hold the largest product, or
// 0 where the step needs the whole row.  A city off the list has a choice
// value of at most M, its tail's largest, and draws r < 1, so its product,
// rounded, is at most M: a listed unvisited city whose product exceeds M beats
// them all, and the list is in city order, so the lowest lane holding the
// largest product is the lowest city.  One Philox block a lane instead of two
// per pass.
__device__ __forceinline__ uint64_t product_list_hit(u32x2 v, bool unvisited, uint32_t k0,
                                                     uint32_t k1, uint32_t step, uint32_t ant,
                                                     uint32_t iter, int lane) {
    const int city = list_city(v.y);
    const uint32_t ctr[1] = {1u + (uint32_t)city / 4u};
    u32x4 x[1];
    philox4_many<1>(k0, k1, step, ant, iter, ctr, x);
    const uint32_t lo = city & 1 ? x[0].y : x[0].x, hi = city & 1 ? x[0].w : x[0].z;
    const float prod = __uint_as_float(v.x) * unit24(city & 2 ? hi : lo);
    const uint32_t key = ((lane < kListEntries) & unvisited) ? __float_as_uint(prod) : 0u;
    const uint32_t top = wave_max_u32(key);
    const uint32_t rest = (uint32_t)__builtin_amdgcn_readlane((int)v.x, kListEntries);
    return top > rest ? ballot(key == top) : 0ull;
}

// The same from the row's wide list, or -1: four Philox blocks a lane.
__device__ __forceinline__ int product_wide_pick(const WideEntries& v, const uint8_t* s_seen,
                                                 uint32_t k0, uint32_t k1, uint32_t step,
                                                 uint32_t ant, uint32_t iter, int lane) {
    uint32_t ctr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) ctr[e] = 1u + (uint32_t)v.city(e) / 4u;
    u32x4 x[4];
    philox4_many<4>(k0, k1, step, ant, iter, ctr, x);
    uint32_t key[4], largest = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int city = v.city(e);
        const uint32_t lo = city & 1 ? x[e].y : x[e].x, hi = city & 1 ? x[e].w : x[e].z;
        const float prod = v.w[e] * unit24(city & 2 ? hi : lo);
        const bool may = (4 * lane + e < kWideEntries) & (s_seen[city] == 0);
        key[e] = may ? __float_as_uint(prod) : 0u;
        largest = max(largest, key[e]);
    }
    const uint32_t top = wave_max_u32(largest);
    const uint32_t rest = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(v.w[3]), 63);
    if (top <= rest) return -1;
    // cities grow with (lane, position)
    int city = 0;
#pragma unroll
    for (int e = 3; e >= 0; --e) city = key[e] == top ? v.city(e) : city;
    return __builtin_amdgcn_readlane(city, __builtin_ctzll(ballot(largest == top)));
}

// Bits of a new tour: cities < n.
template <int P>
__device__ __forceinline__ uint64_t initial_bits(int n, int lane) {
    uint64_t bits = 0;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < kG; ++e)
            if (city_of(p, lane, e) < n) bits |= 1ull << (kG * p + e);
    return bits;
}

// Clears city j's bit in the lane that holds it.
__device__ __forceinline__ void mark_visited(int j, int lane, uint64_t& bits) {
    // j >= 0: unsigned, so the divisions are shifts and masks
    const uint32_t uj = (uint32_t)j;
    const uint32_t p = uj / kPass, rem = uj - p * kPass;
    if ((int)(rem / kG) == lane) bits &= ~(1ull << (kG * p + rem % kG));
}

// Whether colony c's product rule may use the short lists: not where every
// weight is tau^0 / d^0 = 1.  What builds the lists and what reads them ask this.
__host__ __device__ inline bool product_uses_lists(const Colony& c) {
    return c.alpha != 0 || c.beta != 0;
}

template <int P>
__global__ __launch_bounds__(64) void k_construct_product(Colony c, uint32_t iter) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint8_t s_bits[64 * P];
    const int lane = threadIdx.x;
    const int k = ant_of_block(blockIdx.x, c.m);
    const int n = c.n;
    uint16_t* s_tour = reinterpret_cast<uint16_t*>(smem);
    const PhiloxKey key{(uint32_t)c.seed, (uint32_t)(c.seed >> 32)};
    const uint32_t x0 = draw(key, iter, (uint32_t)k, 0u);
    int cur = (int)(((uint64_t)x0 * (uint64_t)(uint32_t)n) >> 32);

    const auto whole_row = [&](int at, int step, uint64_t bits) {
        const PhiloxDraws draws{key.k0, key.k1, (uint32_t)step, (uint32_t)k, iter};
        const uint32_t j =
            product_pick<P>(c.choice + (size_t)at * c.ld, n, bits, draws, lane).city;
        // n - step >= 1 cities are unvisited, so there is one; the clamp only
        // keeps the LDS index in range should that ever break.
        return j == ~0u ? 0 : (int)j;
    };

    if (product_uses_lists(c) && half_by_list(c, kProductRow, lane)) {
        // A step reads its city's short list first, for long rows the wide
        // list where that does not settle the selection, and then the whole
        // row.  Whole rows only -> lists, mean of 20 iterations with m = n: n =
        // 2400 8.56 -> 1.30 ms, n = 1000 0.816 -> 0.400 ms, n = 333 0.177 -> 0.130
        // ms, n = 100 0.0546 -> 0.0459 ms (with the launch that builds the
        // lists, 4 to 15 us).
        uint8_t* s_seen = clear_flags(smem + tour_bytes(n), n, 512 * P, lane);
        const __amdgpu_buffer_rsrc_t lists = list_rsrc(c);
        int step = 1;
        do {
            const u32x2 entry = load_list(lists, cur, lane);
            if (lane == 0) {
                s_tour[step - 1] = (uint16_t)cur;
                s_seen[cur] = 1;
            }
            const uint64_t hit =
                product_list_hit(entry, s_seen[list_city(entry.y)] == 0, key.k0, key.k1,
                                 (uint32_t)step, (uint32_t)k, iter, lane);
            if (__builtin_expect(hit != 0, 1)) {
                cur = list_city(__builtin_amdgcn_readlane(entry.y, __builtin_ctzll(hit)));
            } else {
                int next = -1;
                if constexpr (kPass * (P - 1) >= kMinWideCities)
                    next = product_wide_pick(load_wide(wide_rsrc(c), cur, lane), s_seen, key.k0,
                                             key.k1, (uint32_t)step, (uint32_t)k, iter, lane);
                if (next < 0) {
                    uint64_t bits, blocks;
                    bits_from_flags<P>(reinterpret_cast<const uint2*>(s_seen), s_bits, lane, bits,
                                       blocks);
                    next = whole_row(cur, step, bits);
                }
                cur = next;
            }
            // one city for the wavefront
            cur = __builtin_amdgcn_readfirstlane(cur);
        } while (++step < n);
    } else {
        uint64_t bits = initial_bits<P>(n, lane);
        for (int step = 1; step < n; ++step) {
            if (lane == 0) s_tour[step - 1] = (uint16_t)cur;
            mark_visited(cur, lane, bits);
            cur = __builtin_amdgcn_readfirstlane(whole_row(cur, step, bits));
        }
    }
    if (lane == 0) s_tour[n - 1] = (uint16_t)cur;
    __syncthreads();
    if (lane == 0) s_tour[n] = s_tour[0];
    __syncthreads();

    // Tour length C^k (int64), deposit fl32(1/C^k), tour and neighbour tables.
    long long len = 0;
    for (int s = lane; s < n; s += 64) {
        const int i = s_tour[s], j = s_tour[s + 1];
        len += c.dist[(size_t)i * c.ld + j];
        c.succ[(size_t)i * c.mp + k] = (uint16_t)j;
        c.pred[(size_t)j * c.mp + k] = (uint16_t)i;
    }
    uint16_t* trow = c.tours + (size_t)k * c.tp;
    for (int s = lane; s <= n; s += 64) trow[s] = s_tour[s];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) len += __shfl_xor(len, off);
    if (lane == 0) {
        c.lens[k] = len;
        c.dep[k] = (float)(1.0 / (double)len);
    }
}

template <int P>
__global__ __launch_bounds__(64) void k_test_product_select(const float* rows, int ld, int n,
                                                            const uint8_t* feasible,
                                                            const float* u, int32_t* out) {
    const int lane = threadIdx.x;
    const int q = blockIdx.x;
    const uint8_t* f = feasible + (size_t)q * n;
    uint64_t bits = 0;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < kG; ++e) {
            const int j = city_of(p, lane, e);
            if (j < n && f[j]) bits |= 1ull << (kG * p + e);
        }
    const ArrayDraws draws{u + (size_t)q * n, n};
    const Pick mine = product_pick<P>(rows + (size_t)q * ld, n, bits, draws, lane);
    if (lane == 0) out[q] = mine.city == ~0u ? -1 : (int)mine.city;
}

// Philox throughput probe: the draws of `steps` steps of a 2400-city row
// (ten blocks per lane per step, the formulation construction uses) without
// loads or selection.  The XOR of all words goes to sink[64 * wave + lane].
__global__ __launch_bounds__(64) void k_probe_philox(int steps, uint32_t seed, uint32_t* sink) {
    const int lane = threadIdx.x;
    uint32_t acc = 0;
    for (int step = 1; step <= steps; ++step) {
        uint32_t ctr[10];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const uint32_t q = (uint32_t)(kPass * i + kG * lane) / 4u;
            ctr[2 * i] = 1u + q;
            ctr[2 * i + 1] = 2u + q;
        }
        u32x4 x[10];
        philox4_many<10>(seed, 0u, (uint32_t)step, blockIdx.x, 0u, ctr, x);
#pragma unroll
        for (int i = 0; i < 10; ++i) acc ^= x[i].x ^ x[i].y ^ x[i].z ^ x[i].w;
    }
    sink[(size_t)blockIdx.x * 64 + lane] = acc;
}

// Calls f.template operator()<P>() for P = ceil(n / 512) in 1..8.
template <int P = 1, typename F>
hipError_t dispatch_passes(int n, F&& f) {
    if constexpr (P > kMaxPasses) {
        return hipErrorInvalidValue;
    } else {
        if ((n + kPass - 1) / kPass == P) return f.template operator()<P>();
        return dispatch_passes<P + 1>(n, f);
    }
}

}  // namespace

hipError_t launch_construct_product(const Colony& c, uint32_t iter, hipStream_t s) {
    if (c.n < 1 || c.n > kMaxCities) return hipErrorInvalidValue;
    if (product_uses_lists(c)) {
        const hipError_t e = launch_short_lists(c, s);
        if (e != hipSuccess) return e;
    }
    return dispatch_passes(c.n, [&]<int P>() {
        hipLaunchKernelGGL((k_construct_product<P>), dim3(c.m), dim3(64),
                           tour_bytes(c.n) + seen_lds_bytes(c.n), s, c, iter);
        return hipGetLastError();
    });
}

hipError_t launch_probe_philox(int waves, int steps, uint32_t seed, uint32_t* sink,
                               hipStream_t s) {
    if (waves <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_probe_philox, dim3(waves), dim3(64), 0, s, steps, seed, sink);
    return hipGetLastError();
}

hipError_t launch_test_product_select(int n, int count, const float* rows,
                                      const uint8_t* feasible, const float* u, int32_t* out,
                                      hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (n < 1 || n > kMaxCities) return hipErrorInvalidValue;
    const int ld = (n + 63) & ~63;
    return dispatch_passes(n, [&]<int P>() {
        hipLaunchKernelGGL((k_test_product_select<P>), dim3(count), dim3(64), 0, s, rows,
                           ld, n, feasible, u, out);
        return hipGetLastError();
    });
}

}  // namespace aco
