// construct.hip -- AS tour construction on gfx950 (Section II, Eq. 1; the
// data-parallel design of Section III-A: one workgroup per ant, the ant's
// candidate cities spread over the lanes).
//
// Rows of at most 256 cities (320 at tile 4 and in the batched launch) have a
// layout of their own (construct_flat.hpp).
// Layout of one step of longer rows (ant at city `cur`, wavefront of 64 lanes,
// tile G = 4 or 8 cities per lane):
//   * the choice row of `cur` is streamed with 16-byte loads; in pass p lane l
//     holds cities 64Gp + Gl .. 64Gp + Gl + G-1, so one pass reads 256 G bytes
//     contiguously and every 64-city block sits in 64/G neighbouring lanes;
//   * visited cities are masked to +0 with a per-lane bit set (bit Gp + e);
//     with SKIP, a 16-byte load whose four cities are all visited (or beyond
//     n) is sent to an out-of-range offset instead, which returns zeros
//     without a memory access, so late in a tour the lines of the row that
//     hold no unvisited city are not fetched at all.  That saves bandwidth
//     where the launch is bandwidth-bound (rows of four or more passes at
//     tile 8, and the batched launch) but lengthens a step where it is
//     latency-bound (shorter rows with about one wavefront per SIMD; tile 8
//     takes construct_masked.hpp there), so it is on only in the former;
//   * the total T_b of each 64-city block is a balanced pairwise sum: log2 G
//     levels inside the lane, log2(64/G) DPP levels across the lanes.  That
//     is exactly the last entry of the 64-wide S64 prefix tree, so every T_b
//     is bit-identical to the roulette's definition whatever G is;
//   * T_b move to lane b (a cross-lane read per pass, or for rows of one
//     pass an LDS store and load) and are scanned with S64 (DPP), giving the
//     block offsets E_b and the total;
//   * a block can hold the chosen city only if fl(E_b + T_b (1 + 2^-20)) >
//     target: every inner prefix of a block is at most T_b (1 + 13 u) for a
//     depth-6 tree of non-negative terms (u = 2^-24), so blocks failing this
//     test can be skipped without changing the result;
//   * surviving blocks are rescanned one element per lane with the exact S64
//     tree, in block order, until the first feasible prefix above the target.
// Before any of that, once pheromone has gathered, a step reads only its row's
// short list (shortlist.hpp) and takes the city it proves to be the rule's;
// the steps above then run only where the list does not settle it.
// Random numbers: Philox draws (seed, iter, ant, step), 64 steps at a time on
// the vector unit.
#include <type_traits>

#include "construct_flat.hpp"
#include "construct_masked.hpp"
#include "r64_lanes.hpp"
#include "seen.hpp"
#include "shortlist.hpp"

namespace aco {
namespace {

constexpr int kSkipOffset = 1 << 30;  // past any row: a buffer load there returns 0

// Per-lane feasibility bits: bit G p + e <=> city 64 G p + G lane + e is < n
// and not yet visited.
template <int G, int P>
__device__ __forceinline__ uint64_t initial_lane_bits(int n, int lane) {
    uint64_t bits = 0;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < G; ++e)
            if (p * Tile<G>::kPass + lane * G + e < n) bits |= 1ull << (p * G + e);
    return bits;
}

// The per-lane feasibility bits in 32 bits where P G <= 32 (rows of up to
// 1024 cities), so that clearing one takes 32-bit operations only.
template <int G, int P>
using LaneBits = std::conditional_t<(P * G <= 32), uint32_t, uint64_t>;

// Marks city j visited in both tabu representations (called with j uniform).
template <int G, typename B>
__device__ __forceinline__ void mark_visited(int j, int lane, B& lane_bits,
                                             uint64_t& block_bits) {
    // j >= 0: unsigned, so the divisions are shifts and masks
    const uint32_t uj = (uint32_t)j;
    if (lane == (int)(uj >> 6)) block_bits |= 1ull << (uj & 63);
    const int owner = (int)((uj % Tile<G>::kPass) / G);
    const int bit = (int)((uj / Tile<G>::kPass) * G + (uj % G));
    // a select rather than a branch around the owner lane
    lane_bits &= lane == owner ? ~((B)1 << bit) : ~(B)0;
}

// Stages the masked weights of block `b` into s_w (city 64b + t at s_w[t]).
// The block lives in pass b/G, lanes
// (64/G)(b mod G) .. (64/G)(b mod G + 1) - 1; the pass index is wave-uniform
// but not a compile-time constant, so each pass has its own branch, and the
// stores are opaque to the optimiser so that it cannot merge the branches
// into per-register selects.
template <int G, int P>
__device__ __forceinline__ void stage_block(const u32x4 (&wa)[P], const u32x4 (&wb)[P], int b,
                                            float* s_w, int lane) {
    const int pb = b / G;
    if (lane / Tile<G>::kLanesPerBlock != (b % G)) return;
    const uint32_t addr = (uint32_t)(uintptr_t)(s_w + lane % Tile<G>::kLanesPerBlock * G);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (p == pb) {
            if (G == 8)
                asm volatile("ds_write_b128 %0, %1\n\tds_write_b128 %0, %2 offset:16"
                             :
                             : "v"(addr), "v"(wa[p]), "v"(wb[p])
                             : "memory");
            else
                asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(wa[p]) : "memory");
        }
    }
}

// Issues the loads of row `row` of the ld-padded matrix `mat` into wa/wb:
// in pass p lane l takes cities 64Gp + Gl .. + G - 1.  The descriptor
// spans `records` bytes from mat and stays the same for the whole tour; the
// row is selected by the scalar offset (two scalar operations per step), and
// the range check covers scalar plus vector offset.  Loads past the end of
// the span return zeros without touching memory; those past the row's n
// cities but inside the span read padding or the next row, and masking
// (whose bits exist only for cities < n) zeroes them.  With SKIP, a 16-byte
// load whose four cities are all visited goes out of range instead.
// With FEW, at most six loads are in flight: a load waits until all but two of
// those before it have returned.
template <int G, int P, bool SKIP, bool FEW = false, typename B>
__device__ __forceinline__ void load_row(const float* __restrict__ mat, int records, int row,
                                         int row_bytes, B lane_bits, int lane, u32x4 (&wa)[P],
                                         u32x4 (&wb)[P]) {
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(mat, records);
    const int soff = row * row_bytes;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t bits = (uint32_t)(lane_bits >> (p * G));
        const int off = (p * Tile<G>::kPass + lane * G) * 4;
        if (FEW && p >= 2) asm volatile("s_waitcnt vmcnt(2)" : : : "memory");
        const int oa = (!SKIP || (bits & 0xFu)) ? off : kSkipOffset;
        wa[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, oa, soff, 0);
        if (G == 8) {
            const int ob = (!SKIP || (bits & 0xF0u)) ? off + 16 : kSkipOffset;
            wb[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, ob, soff, 0);
        }
    }
}

// Whole rows in LDS: after masking, every pass's weights go to s_w (city c at
// s_w[c]), so that a candidate block is read back with one load and nothing is
// staged on the way to the selection.  Otherwise the masked weights stay in
// registers and only a candidate block is staged.  Rows of one pass are stored
// whole everywhere, rows of up to 1024 cities with ALL: where the launch is
// bound by latency.  The 4 KB an ant that ALL takes leave room for fewer ants on a
// compute unit where there are many.  All / block, whole rows: one batched
// instance of 1000 cities 0.59 / 0.63 ms, four of 600 0.52 / 0.54, eight of 700 1.47 /
// 1.23, 10 of 600 1.14 / 1.03; n = 1000 with 8192 ants 1.96 / 1.70.
template <int G, int P, bool ALL>
constexpr bool kWriteAllPasses = (P * Tile<G>::kPass <= (ALL ? 1024 : 512));

// Two passes: both passes' masks and lane sums before either's sums across
// lanes (left to itself, the compiler finishes one pass and waits for its
// cross-lane read before the next: n = 1000 with 4096 ants 0.945 against 0.924
// ms; no difference in batches).
template <int P>
constexpr bool kTogether = P == 2;

// Lane b of T takes the total of block b of pass p from t, whose groups' last
// lanes hold the pass's block totals.
template <int G>
__device__ __forceinline__ float to_blocks(float t, int p, float T, int lane) {
    constexpr int LPB = Tile<G>::kLanesPerBlock;
    const float x = __int_as_float(__builtin_amdgcn_ds_bpermute(
        ((lane % G) * LPB + LPB - 1) * 4, __float_as_int(t)));
    return lane / G == p ? x : T;
}

// One R64 roulette draw over a loaded row of P passes (wa/wb as load_row
// leaves them; masked in place).  block_bits: the visited bits of block b in
// lane b.  Returns the chosen city, or -1 if no city is feasible.
// Wave-uniform.  The workgroup is one wavefront: its LDS operations execute
// in program order, and every LDS access below uses a lane-dependent index,
// so the compiler keeps the order.
template <int G, int P, bool ALL, typename B>
__device__ __forceinline__ int pick_loaded(u32x4 (&wa)[P], u32x4 (&wb)[P], int n, B lane_bits,
                                           uint64_t block_bits, float* s_T, float* s_w, float u,
                                           int lane) {
    constexpr int LPB = Tile<G>::kLanesPerBlock;
    constexpr bool kAll = kWriteAllPasses<G, P, ALL>;
    // Block totals to lane b (0 past the row's blocks).  Rows of two or more
    // passes fetch them with one cross-lane read per pass from the last lane
    // of each group (and rows staged whole store their weights afterwards):
    // against a masked LDS store per pass and a load, n = 2400 0.8% faster, and
    // batched one instance of 700 cities 0.395 against 0.434 ms, of 1000 0.591
    // against 0.620, of 1500 1.46 against 1.50.  Rows of one pass keep the
    // store and load (cross-lane reads measured 6% slower at n = 512).
    constexpr bool kPermute = P >= 2;
    const int nb = (n + 63) >> 6;
    float T = 0.0f;
    float part[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t bits = (uint32_t)(lane_bits >> (p * G));
        mask4<0>(wa[p], bits);
        if (G == 8) {
            mask4<4>(wb[p], bits);
            part[p] = pair_sum4(wa[p]) + pair_sum4(wb[p]);
        } else {
            part[p] = pair_sum4(wa[p]);
        }
        if (!kPermute) {
            if (kAll) {
                u32x4* dst = reinterpret_cast<u32x4*>(s_w + p * Tile<G>::kPass + lane * G);
                dst[0] = wa[p];
                if (G == 8) dst[1] = wb[p];
            }
            const float t = group_pairwise<LPB>(part[p]);
            if ((lane % LPB) == LPB - 1) s_T[p * G + lane / LPB] = t;
        } else if (!kTogether<P>) {
            T = to_blocks<G>(group_pairwise<LPB>(part[p]), p, T, lane);
        }
    }
    if (kPermute) {
        if (kTogether<P>) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < P; ++p) part[p] = group_pairwise<LPB>(part[p]);
#pragma unroll
            for (int p = 0; p < P; ++p) T = to_blocks<G>(part[p], p, T, lane);
            __builtin_amdgcn_sched_barrier(0x7F);  // no LDS store above the reads
        }
        if (kAll) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                u32x4* dst = reinterpret_cast<u32x4*>(s_w + p * Tile<G>::kPass + lane * G);
                dst[0] = wa[p];
                if (G == 8) dst[1] = wb[p];
            }
        }
    } else {
        T = s_T[lane];
    }
    // Rows of at most 1024 cities have nb <= 16 blocks, all in row 0 of the
    // block-total scan, which stage B leaves as it is; rows of at most 2^L
    // blocks need only its first L levels.
    float I;
    if constexpr (P * G <= 16)
        I = s64_scan_row0_levels<block_scan_levels(P * G)>(T);
    else
        I = s64_scan(T);
    const float total = read_lane(I, nb - 1);
    const float target = u * total;
    const float E = wave_shift_up1(I);
    const float bound = E + T * kBlockSlack;
    uint64_t cand = ballot(bound > target) & (nb >= 64 ? ~0ull : (1ull << nb) - 1ull);
    // Nearly always exactly one candidate block: a single-exit loop, tested
    // at the bottom, so that the usual step runs through without a taken
    // branch.  It goes on while `more` (the remaining candidates, or 0 once
    // the city is found) is not 0, made opaque so that the test stays one
    // compare of a register pair.
    int j = -1;
    if (__builtin_expect(cand != 0, 1)) {
        uint64_t more;
        do {
            const int b = __builtin_ctzll(cand);
            cand &= cand - 1;
            float w;
            if (kAll) {
                w = s_w[b * 64 + lane];
            } else {
                stage_block<G, P>(wa, wb, b, s_w, lane);
                w = s_w[lane];
            }
            const uint64_t vis = lane_u64(block_bits, b);
            const float s = s64_scan(w);
            const float eb = read_lane(E, b);
            const uint64_t hit = ballot((eb + s) > target) & ~vis;
            if (hit) j = b * 64 + __builtin_ctzll(hit);
            more = hit != 0 ? 0ull : cand;
            __asm__("" : "+s"(more));
        } while (__builtin_expect(more != 0, 0));
    }
    if (__builtin_expect(j >= 0, 1)) return j;
    return pick_fallback(block_bits);
}

template <int G, int P, bool SKIP, bool ALL, typename B>
__device__ __forceinline__ int r64_pick(const float* __restrict__ mat, int records, int row,
                                        int row_bytes, int n, B lane_bits, uint64_t block_bits,
                                        float* s_T, float* s_w, float u, int lane) {
    u32x4 wa[P], wb[P];
    load_row<G, P, SKIP>(mat, records, row, row_bytes, lane_bits, lane, wa, wb);
    return pick_loaded<G, P, ALL>(wa, wb, n, lane_bits, block_bits, s_T, s_w, u, lane);
}

// LDS a construction workgroup needs besides the tour and the visited flags.
template <int W>
struct AntShared {
    float w[W];   // masked weights of whole rows, or a staged block
    float T[64];  // block totals in block order
};

// Words that a kernel for rows of P passes stages: whole rows, or a block and the
// 64 P bytes that bits_from_flags uses (with a whole pass staged, an ant of 3500
// cities took an LDS granule more, and m = n = 3500 two rounds: 22.1 against 20.6
// ms on whole rows).
template <int G, int P, bool ALL>
constexpr int kStaged = kWriteAllPasses<G, P, ALL> ? P * Tile<G>::kPass : 128;
static_assert(64 * (kMaxCities / 512) <= 128 * sizeof(float), "bits_from_flags' scratch");

// Tiles whose colonies use the short lists (uses_lists).
template <int G>
constexpr bool kUseLists = G == 8;

// Whether every row of P passes has a wide list.
template <int G, int P>
constexpr bool kWideLists = 64 * G * (P - 1) >= kMinWideCities;

// Dynamic LDS of an ant: the tour, then the flags.
__host__ __device__ size_t ant_lds_bytes(int n) { return tour_lds_bytes(n) + seen_lds_bytes(n); }

// Staging of the batched launch's kernel, which serves rows of any length.
template <bool ALL>
constexpr int kBatchStaged = ALL ? 1024 : 512;

// Whether the flags of P passes lie in AntShared<W>::w behind what the ant stages
// there: in the batched launch, where short and long rows share W, so that
// rows of several lengths ask for no more LDS than their tour (n = 2400: 16 ants a
// compute unit against 12).
template <int G, int P, bool ALL, int W>
constexpr bool kFlagsInStaging = W * sizeof(float) >=
                                 kStaged<G, P, ALL> * sizeof(float) + 512 * P;

// Dynamic LDS of an ant of n cities in the batched launch.
template <bool ALL>
size_t batch_ant_lds_bytes(int n) {
    constexpr int W = kBatchStaged<ALL>;
    const bool behind[] = {kFlagsInStaging<8, 1, ALL, W>, kFlagsInStaging<8, 2, ALL, W>,
                           kFlagsInStaging<8, 3, ALL, W>, kFlagsInStaging<8, 4, ALL, W>,
                           kFlagsInStaging<8, 5, ALL, W>, kFlagsInStaging<8, 6, ALL, W>,
                           kFlagsInStaging<8, 7, ALL, W>, kFlagsInStaging<8, 8, ALL, W>};
    const bool flags =
        n <= 64 * kMaxFlatBlocks ? n > kMinListCities : !behind[(n + 511) / 512 - 1];
    return tour_lds_bytes(n) + (flags ? seen_lds_bytes(n) : 0);
}

// The same for any ant of up to max_n cities: the largest of each layout and
// pass count.
template <bool ALL>
size_t batch_ants_lds_bytes(int max_n) {
    size_t most = batch_ant_lds_bytes<ALL>(max_n < 64 * kMaxFlatBlocks ? max_n
                                                                       : 64 * kMaxFlatBlocks);
    for (int n = 512; n < max_n + 512; n += 512) {
        const size_t need = batch_ant_lds_bytes<ALL>(n < max_n ? n : max_n);
        most = need > most ? need : most;
    }
    return most;
}

// The same for an ant that keeps the visited set as factors.
__host__ __device__ size_t masked_lds_bytes(int n) {
    return tour_lds_bytes(n) + seen_lds_bytes(n) * sizeof(float);
}

// Whether the roulette of colony c starts its steps from the short lists:
// where half of the rows have a list that covers them well.
__device__ __forceinline__ bool starts_from_lists(const Colony& c, int lane) {
    return uses_lists(c) && half_by_list(c, kRouletteRow, lane);
}

// The end of a tour: its last city `cur`, then length, deposit, tour and
// neighbour tables.
__device__ __forceinline__ void finish_ant(const Colony& c, int k, int cur, uint16_t* s_tour,
                                           int lane) {
    const int n = c.n;
    // one wavefront's LDS operations execute in program order
    if (lane == 0) s_tour[n - 1] = (uint16_t)cur;
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) s_tour[n] = s_tour[0];
    __builtin_amdgcn_wave_barrier();

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


// The n - 1 selections of ant k from its start city: step(cur, u, i) is the
// next city of the i-th (0 .. n - 2).  64 steps at a time: their draws come
// from one Philox call on the vector unit, and with KEEP the cities left go
// to a register, one lane a step, and from there to s_tour at once (three
// instructions a step; a store by one lane takes six).  Returns the last city.
template <bool KEEP, typename Step>
__device__ __forceinline__ int walk(int n, PhiloxKey key, uint32_t iter, int k, uint16_t* s_tour,
                                    int lane, Step&& step) {
    const uint32_t x0 = draw(key, iter, (uint32_t)k, 0u);
    int cur = (int)(((uint64_t)x0 * (uint64_t)(uint32_t)n) >> 32);
    for (int base = 0; base < n - 1; base += 64) {
        const float u64 = draws64(key, iter, (uint32_t)k, base + 1, lane);
        const int count = __builtin_amdgcn_readfirstlane(n - 1 - base < 64 ? n - 1 - base : 64);
        uint32_t left = 0;
        int t = 0;
        do {
            if (KEEP) left = lane == t ? (uint32_t)cur : left;
            // one city for the wavefront; taken as per-lane, every row load
            // of the next step would become a loop over lanes
            cur = __builtin_amdgcn_readfirstlane(step(cur, read_lane(u64, t), base + t));
        } while (++t < count);
        if (KEEP && lane < count) s_tour[base + lane] = (uint16_t)left;
    }
    return cur;
}

// The whole tour of ant k for rows of at most B blocks of 64 cities.
template <int B, bool LIST>
__device__ __forceinline__ void construct_ant_flat(const Colony& c, int k, uint32_t iter,
                                                   uint16_t* s_tour, int lane) {
    const int n = c.n;
    const int row_bytes = c.ld * 4, records = n * row_bytes;
    const PhiloxKey key{(uint32_t)c.seed, (uint32_t)(c.seed >> 32)};
    Unvisited<B> live(n);
    int cur;
    bool by_list = false;
    if constexpr (LIST) by_list = starts_from_lists(c, lane);
    if (LIST && by_list) {
        // as in construct_ant
        const __amdgpu_buffer_rsrc_t lists = list_rsrc(c);
        uint8_t* s_seen = clear_flags(reinterpret_cast<uint8_t*>(s_tour) + tour_lds_bytes(n), n, 512, lane);
        cur = walk<false>(n, key, iter, k, s_tour, lane, [&](int at, float u, int i) {
            const u32x2 entry = load_list(lists, at, lane);
            if (lane == 0) {
                s_tour[i] = (uint16_t)at;
                s_seen[at] = 1;
            }
            const bool unvisited = s_seen[list_city(entry.y)] == 0;
            const uint64_t hit = roulette_list_hit(entry, list_weight(entry, unvisited, lane), u);
            if (__builtin_expect(hit != 0, 1)) return hit_city(entry, hit);
            uint32_t x[B];
            load_flat<B>(c.choice, records, at, row_bytes, lane, x);
            live.from_flags(s_seen, lane);
            return pick_flat<B>(x, live, u);
        });
    } else {
        cur = walk<true>(n, key, iter, k, s_tour, lane, [&](int at, float u, int) {
            uint32_t x[B];
            load_flat<B>(c.choice, records, at, row_bytes, lane, x);
            live.visit(at, lane);
            return pick_flat<B>(x, live, u);
        });
    }
    finish_ant(c, k, cur, s_tour, lane);
}

// LDS of a masked ant: the row as loaded and its block totals.
template <int P>
struct MaskedShared {
    float w[512 * P];
    float T[64];
};

// The whole tour of ant k for rows of P passes of 512 cities, P <= 3.
template <int P>
__device__ __forceinline__ void construct_ant_masked(const Colony& c, int k, uint32_t iter,
                                                     uint16_t* s_tour, float* s_w, float* s_T,
                                                     int lane) {
    const int n = c.n;
    const int row_bytes = c.ld * 4, records = n * row_bytes;
    const PhiloxKey key{(uint32_t)c.seed, (uint32_t)(c.seed >> 32)};
    float* s_f = reinterpret_cast<float*>(reinterpret_cast<char*>(s_tour) + tour_lds_bytes(n));
    init_factors<P>(s_f, n, lane);
    s_T[lane] = 0.0f;
    int cur;
    if (starts_from_lists(c, lane)) {
        // As in construct_ant; the factors serve both kinds of step.  m = n,
        // with the lists' launch against whole rows with the bits, in the
        // 20th iteration: n = 500 0.136 / 0.197 ms, n = 1000 0.285 / 0.508, n =
        // 1500 0.496 / 1.31; mean of the first 24: 0.157 / 0.198, 0.363 /
        // 0.519, 0.791 / 1.32.
        const __amdgpu_buffer_rsrc_t lists = list_rsrc(c);
        cur = walk<false>(n, key, iter, k, s_tour, lane, [&](int at, float u, int i) {
            const u32x2 entry = load_list(lists, at, lane);
            if (lane == 0) {
                s_tour[i] = (uint16_t)at;
                s_f[at] = 0.0f;
            }
            const float w = __uint_as_float(entry.x) * s_f[list_city(entry.y)];
            const uint64_t hit = roulette_list_hit(entry, lane < kListEntries ? w : 0.0f, u);
            if (__builtin_expect(hit != 0, 1)) return hit_city(entry, hit);
            u32x4 wa[P], wb[P];
            load_passes<P>(c.choice, records, at, row_bytes, lane, wa, wb);
            const int j = pick_masked<P>(wa, wb, n, s_f, s_T, s_w, u, lane);
            return j < 0 ? 0 : j;
        });
    } else {
        cur = walk<true>(n, key, iter, k, s_tour, lane, [&](int at, float u, int) {
            u32x4 wa[P], wb[P];
            load_passes<P>(c.choice, records, at, row_bytes, lane, wa, wb);
            if (lane == 0) s_f[at] = 0.0f;
            const int j = pick_masked<P>(wa, wb, n, s_f, s_T, s_w, u, lane);
            return j < 0 ? 0 : j;
        });
    }
    finish_ant(c, k, cur, s_tour, lane);
}

template <int P>
__global__ __launch_bounds__(64) void k_construct_masked(Colony c, uint32_t iter) {
    extern __shared__ __align__(16) uint16_t s_tour[];
    __shared__ __align__(16) MaskedShared<P> sh;
    construct_ant_masked<P>(c, ant_of_block(blockIdx.x, c.m), iter, s_tour, sh.w, sh.T,
                            threadIdx.x);
}

template <int B>
__global__ __launch_bounds__(64) void k_construct_flat(Colony c, uint32_t iter) {
    extern __shared__ __align__(16) uint16_t s_tour[];
    construct_ant_flat<B, (64 * B > kMinListCities)>(c, ant_of_block(blockIdx.x, c.m), iter,
                                                     s_tour, threadIdx.x);
}

// Rows of five passes and more, read whole, are loaded in one burst where the
// launch is bound by latency, and with few loads in flight where it is bound by
// memory (more rows in flight then only displace one another from the caches).
// One burst / few, alpha 0, beta 1: n = 2400, m = 1024 2.80 / 3.17 ms, m = 2048 5.15 /
// 5.20, m = 2400 6.16 / 5.93; n = 3000, m = 1400 5.88 / 5.85, m = 2000 8.5 / 8.3; n =
// 4096, m = 1000 8.18 / 8.22, m = 1500 13.4 / 12.2.
constexpr int kMinFewPasses = 5;
__device__ __forceinline__ bool memory_bound(const Colony& c) { return c.m * c.n >= 5000000; }

// The whole tour of ant k of colony c in iteration `iter`: placement, n - 1
// roulette steps, then length, deposit, tour and neighbour tables.
template <int G, int P, bool SKIP, bool LOAD_FIRST, bool LIST, bool ALL, int W>
__device__ __forceinline__ void construct_ant(const Colony& c, int k, uint32_t iter,
                                              uint16_t* s_tour, AntShared<W>& sh) {
    const int lane = threadIdx.x;
    const int n = c.n;
    const int records = n * c.ld * 4;  // the whole n x ld choice matrix
    const PhiloxKey key{(uint32_t)c.seed, (uint32_t)(c.seed >> 32)};

    const int row_bytes = c.ld * 4;
    uint64_t block_bits = initial_block_bits(n, lane);
    sh.T[lane] = 0.0f;
    LaneBits<G, P> lane_bits = (LaneBits<G, P>)initial_lane_bits<G, P>(n, lane);
    __builtin_amdgcn_wave_barrier();

    // LOAD_FIRST: a step's row loads go out as soon as its city is known, and
    // the bookkeeping of that city (tour entry, visited bits) is done while
    // they are in flight.  That shortens steps of one to three passes (with
    // this layout alone: n = 1000 7%, n = 1500 4% faster) but made the
    // bandwidth-bound four- and five-pass launches (n = 2048, 2400) no
    // faster or up to 1% slower, which keep the bookkeeping first.  With
    // LOAD_FIRST the loads see the visited bits without the step's own city;
    // with SKIP that only loads a quad once more, and masking (which sees
    // it) zeroes the city.
    int cur;
    bool by_list = false;
    if constexpr (LIST) by_list = starts_from_lists(c, lane);
    if (LIST && by_list) {
        // A step reads its city's short list, and the whole row only where
        // the list does not settle the selection.  The usual step keeps the
        // flags only; the general step's bits are made from them.  m = n,
        // construction with the lists' launch against whole rows only, in
        // the 20th iteration: n = 2400 1.10 / 6.05 ms, n = 3000 1.68 / 13.3;
        // mean of the first 24: 2.61 / 6.05, 5.10 / 13.2.
        const __amdgpu_buffer_rsrc_t lists = list_rsrc(c);
        uint8_t* s_seen = clear_flags(
            kFlagsInStaging<G, P, ALL, W> ? reinterpret_cast<uint8_t*>(sh.w + kStaged<G, P, ALL>)
                                     : reinterpret_cast<uint8_t*>(s_tour) + tour_lds_bytes(n),
            n, 512 * P, lane);
        cur = walk<false>(n, key, iter, k, s_tour, lane, [&](int at, float u, int i) {
            const u32x2 entry = load_list(lists, at, lane);
            if (lane == 0) {
                s_tour[i] = (uint16_t)at;
                s_seen[at] = 1;
            }
            const bool unvisited = s_seen[list_city(entry.y)] == 0;
            const uint64_t hit = roulette_list_hit(entry, list_weight(entry, unvisited, lane), u);
            if (__builtin_expect(hit != 0, 1)) return hit_city(entry, hit);
            if constexpr (kWideLists<G, P>) {
                if (wide_tried(entry)) {
                    const int j = roulette_wide_pick(load_wide(wide_rsrc(c), at, lane), s_seen, u, lane);
                    if (j >= 0) return j;
                }
            }
            bits_from_flags<P>(reinterpret_cast<const uint2*>(s_seen),
                               reinterpret_cast<uint8_t*>(sh.w), lane, lane_bits, block_bits);
            const int j = r64_pick<G, P, SKIP, ALL>(c.choice, records, at, row_bytes, n, lane_bits,
                                               block_bits, sh.T, sh.w, u, lane);
            return j < 0 ? 0 : j;
        });
    } else {
        const auto whole_rows = [&]<bool FEW>() {
            cur = walk<true>(n, key, iter, k, s_tour, lane, [&](int at, float u, int) {
                u32x4 wa[P], wb[P];
                if (LOAD_FIRST)
                    load_row<G, P, SKIP, FEW>(c.choice, records, at, row_bytes, lane_bits, lane,
                                              wa, wb);
                mark_visited<G>(at, lane, lane_bits, block_bits);
                if (!LOAD_FIRST)
                    load_row<G, P, SKIP, FEW>(c.choice, records, at, row_bytes, lane_bits, lane,
                                              wa, wb);
                const int j = pick_loaded<G, P, ALL>(wa, wb, n, lane_bits, block_bits, sh.T, sh.w,
                                                     u, lane);
                // At every step at least one city is unvisited, so j >= 0; the
                // clamp only keeps the LDS indices in range should that ever
                // break.
                return j < 0 ? 0 : j;
            });
        };
        if (P >= kMinFewPasses && memory_bound(c))
            whole_rows.template operator()<(P >= kMinFewPasses)>();
        else
            whole_rows.template operator()<false>();
    }
    finish_ant(c, k, cur, s_tour, lane);
}

// Tile 8 with up to three passes comes here with many ants only (masked_rows).
template <int G, int P>
__global__ __launch_bounds__(64) void k_construct(Colony c, uint32_t iter) {
    extern __shared__ __align__(16) uint16_t s_tour[];
    constexpr bool kAll = G == 4;
    __shared__ __align__(16) AntShared<kStaged<G, P, kAll>> sh;
    construct_ant<G, P, (P >= 3), (P < 4), kUseLists<G>, kAll>(c, ant_of_block(blockIdx.x, c.m), iter,
                                                         s_tour, sh);
}

// Batched construction: workgroup g builds ant (antmap[g] & 0xffff) of colony
// cols[antmap[g] >> 16] in that colony's current iteration (*iter_dev).  Each
// colony carries its own tile, and its pass count picks the ant's code
// (batch_ant).  P8 bounds the passes of tile-8 colonies (every colony of the
// launch has n <= 512 P8), so a batch of small instances holds no registers
// for rows it does not have; tile 4 is only ever set for n <= 1024 (4
// passes).
// Loads first in the batched launch too, for rows of one to three passes (as
// in the single-instance launch): 757 -> 764 solves/s on the 256-instance
// workload (n 50..1000, same box).  Longer rows keep the bookkeeping first,
// which is no slower where construction is bound by memory.
template <int NP>
constexpr bool kBatchLoadFirst = NP < 4;

// Rows of one to three passes keep the bits here, which skip the loads of
// visited quads, and not the factors of the single-instance launch: with
// those, 64 instances of 50 to 1000 cities took 70.4 ms against 66.1, ten
// served requests 243 against 229 (more LDS an ant, and no load skipped where
// thousands of ants share the L2).
// The ant's code for its colony's exact pass count NP (1 .. PMAX): each
// instance runs a loop specialised for its row length, with no per-pass
// test of the pass count inside the step (256 instances, n 50..1000: 757 ->
// 762 solves/s against one loop with run-time pass tests).
template <int G, int NP, int PMAX, bool ALL, int W>
__device__ __forceinline__ void batch_ant(const Colony& c, int k, uint32_t iter, int np,
                                          uint16_t* s_tour, AntShared<W>& sh) {
    if constexpr (NP < PMAX) {
        if (np != NP) {
            batch_ant<G, NP + 1, PMAX, ALL>(c, k, iter, np, s_tour, sh);
            return;
        }
    }
    construct_ant<G, NP, true, kBatchLoadFirst<NP>, kUseLists<G>, ALL>(c, k, iter, s_tour, sh);
}

template <int B>
__device__ __forceinline__ void batch_ant_flat(const Colony& c, int k, uint32_t iter,
                                               uint16_t* s_tour) {
    if constexpr (B < kMaxFlatBlocks) {
        if (__builtin_amdgcn_readfirstlane(c.n) > 64 * B) {
            batch_ant_flat<B + 1>(c, k, iter, s_tour);
            return;
        }
    }
    construct_ant_flat<B, (64 * B > kMinListCities)>(c, k, iter, s_tour, threadIdx.x);
}

// Rows of up to two passes keep to the scalar registers that eight wavefronts a
// SIMD leave (asked for seven, the compiler stays below; asked for eight, it
// makes the steps 1% longer; with a block of registers more, 16 instances of 400
// cities take two rounds, 0.595 ms against 0.512).
template <int P8, bool ALL>
__global__ __launch_bounds__(64, P8 == 2 ? 7 : 1) void k_construct_batch(const Colony* __restrict__ cols,
                                                        const uint32_t* __restrict__ antmap) {
    extern __shared__ __align__(16) uint16_t s_tour[];
    __shared__ __align__(16) AntShared<kBatchStaged<ALL>> sh;
    const uint32_t e = antmap[blockIdx.x];
    const Colony c = cols[e >> 16];
    // One value for the whole workgroup.  Read through a pointer the kernel
    // might write, it would otherwise be taken as per-lane, and with it the
    // start city and every row address of the tour, each load of which then
    // becomes a loop over lanes.
    const uint32_t iter = __builtin_amdgcn_readfirstlane(*c.iter_dev);
    const int k = (int)(e & 0xffffu);
    if (c.n <= 64 * kMaxFlatBlocks) {
        batch_ant_flat<1>(c, k, iter, s_tour);
    } else if (c.tile == 4) {
        const int np = __builtin_amdgcn_readfirstlane((c.n + 255) / 256);
        batch_ant<4, 2, 4, ALL>(c, k, iter, np, s_tour, sh);
    } else {
        const int np = __builtin_amdgcn_readfirstlane((c.n + 511) / 512);
        batch_ant<8, 1, P8, ALL>(c, k, iter, np, s_tour, sh);
    }
}

template <int G, int P, bool ALL>
__global__ __launch_bounds__(64) void k_test_select(const float* rows, int ld, int n,
                                                     const uint8_t* feasible, const float* us,
                                                     int32_t* out) {
    __shared__ __align__(16) AntShared<kStaged<G, P, ALL>> sh;
    const int lane = threadIdx.x;
    const int q = blockIdx.x;
    const uint8_t* f = feasible + (size_t)q * n;
    uint64_t vis = ~0ull;
    for (int t = 0; t < 64; ++t) {
        const int j = lane * 64 + t;
        if (j < n && f[j]) vis &= ~(1ull << t);
    }
    sh.T[lane] = 0.0f;
    uint64_t lane_bits = 0;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < G; ++e) {
            const int j = p * Tile<G>::kPass + lane * G + e;
            if (j < n && f[j]) lane_bits |= 1ull << (p * G + e);
        }
    __syncthreads();
    // one row per query: the span is that row's n cities (rounded up to whole
    // 16-byte loads; the caller's padding columns are zero)
    const int j = r64_pick<G, P, true, ALL>(rows + (size_t)q * ld, ((n + 3) & ~3) * 4, 0, ld * 4, n,
                                       lane_bits, vis, sh.T, sh.w, us[q], lane);
    if (lane == 0) out[q] = j;
}

template <int P>
__global__ __launch_bounds__(64) void k_test_select_masked(const float* rows, int ld, int n,
                                                           const uint8_t* feasible,
                                                           const float* us, int32_t* out) {
    __shared__ __align__(16) MaskedShared<P> sh;
    __shared__ __align__(16) float s_f[512 * P];
    const int lane = threadIdx.x;
    const int q = blockIdx.x;
    const uint8_t* f = feasible + (size_t)q * n;
    for (int j = lane; j < 512 * P; j += 64) s_f[j] = j < n && f[j] ? 1.0f : 0.0f;
    sh.T[lane] = 0.0f;
    __syncthreads();
    u32x4 wa[P], wb[P];
    load_passes<P>(rows + (size_t)q * ld, ((n + 3) & ~3) * 4, 0, ld * 4, lane, wa, wb);
    // The factors mask by multiplication, which an infinity or a NaN passes.
    // Choice rows hold neither; a row given here may, where it is not feasible.
#pragma unroll
    for (int p = 0; p < P; ++p) {
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            bits |= s_f[512 * p + 8 * lane + e] != 0.0f ? 1u << e : 0u;
        mask4<0>(wa[p], bits);
        mask4<4>(wb[p], bits);
    }
    const int j = pick_masked<P>(wa, wb, n, s_f, sh.T, sh.w, us[q], lane);
    if (lane == 0) out[q] = j;
}

template <int B>
__global__ __launch_bounds__(64) void k_test_select_flat(const float* rows, int ld, int n,
                                                         const uint8_t* feasible, const float* us,
                                                         int32_t* out) {
    const int lane = threadIdx.x;
    const int q = blockIdx.x;
    const uint8_t* f = feasible + (size_t)q * n;
    Unvisited<B> live(n);
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int j = 64 * b + lane;
        live.word[b] = ballot(j < n && f[j] != 0);
    }
    uint32_t x[B];
    load_flat<B>(rows + (size_t)q * ld, n * 4, 0, ld * 4, lane, x);
    const int j = pick_flat<B>(x, live, us[q]);
    if (lane == 0) out[q] = j;
}

// Batched launches can hold at most `wg_per_cu` workgroups on a compute unit
// by asking for more dynamic LDS than the tour needs.  Each workgroup keeps
// one choice row in flight; with more of them the rows evict one another
// from the L2 of each XCD, with fewer the latency of a step is no longer
// covered.  The cap is part of a batch's launch configuration, chosen by the
// batch autotuner; the default (used by the server) caps at 16 per CU, the
// best on a 256-instance batch (n 50..1000; mean of a new and a converged
// state 9.28 ms an iteration, 20 to 32 and no cap 9.29 to 9.33, 12 9.65, 8 11.2;
// where whole rows are read alone, 18 and 20 were 0.7% slower, 24 2.5%, no
// cap 8.7%), and only launches of at least kCapRounds rounds at the cap: one that fits the
// device in a round or two would only gain a tail.
constexpr int kBatchWgPerCu = 16;
constexpr int kCapRounds = 8;

constexpr int kComputeUnits = 256;

// Whether a launch of `ants` ants keeps whole rows in LDS (kWriteAllPasses).
bool whole_rows_in_lds(int ants) { return ants <= 12 * kComputeUnits; }

}  // namespace

size_t batch_lds_bytes(int max_n, int total_ants, int wg_per_cu, size_t lds_per_cu) {
    const bool all = whole_rows_in_lds(total_ants);
    const size_t tour = all ? batch_ants_lds_bytes<true>(max_n) : batch_ants_lds_bytes<false>(max_n);
    if (wg_per_cu <= 0 || lds_per_cu == 0) return tour;
    const size_t per_wg = lds_per_cu / (size_t)wg_per_cu;
    // static LDS and its alignment
    const size_t fixed = (all ? sizeof(AntShared<kBatchStaged<true>>)
                              : sizeof(AntShared<kBatchStaged<false>>)) + 64;
    const size_t cap = per_wg > fixed ? (per_wg - fixed) & ~(size_t)255 : 0;
    return tour > cap ? tour : cap;
}

int batch_default_cap(int total_ants, int cus) {
    return total_ants >= kCapRounds * kBatchWgPerCu * cus ? kBatchWgPerCu : 0;
}

namespace {

// Whether rows of n cities at tile 8 keep the visited set as factors
// (construct_masked.hpp) in a launch of m ants: where the ants fit the device
// in one round.  An ant of P passes then holds 4 KB of LDS a pass beside its
// tour, so that 16 (P = 1, 2) or 9 (P = 3) fit a compute unit, against 28 and
// more with the bits.  First iteration, factors / bits: n = 1000, m = 1000 0.492 /
// 0.511 ms, 2560 0.704 / 0.733, 3500 0.946 / 0.865, 4096 1.27 / 0.91, 16384 3.91 /
// 2.96; n = 1500, m = 1500 1.22 / 1.37, 2048 1.42 / 1.48, 2560 2.44 / 1.73.  Rows
// of one pass are shorter with factors at any m (n = 512, m = 512 0.188 / 0.218,
// 32768 2.02 / 2.08).
bool masked_rows(int n, int m) {
    const int passes = (n + 511) / 512;
    return passes == 1 || (passes <= kMaxMaskedPasses && m <= 24 / passes * kComputeUnits);
}

template <int B = 1, typename F>
hipError_t dispatch_flat(int n, F&& f) {
    if constexpr (B > kMaxFlatBlocks) {
        return hipErrorInvalidValue;
    } else {
        if (n > 64 * B) return dispatch_flat<B + 1>(n, f);
        return f.template operator()<0, B>();
    }
}

template <int G, int P>
auto test_select_kernel(bool all) {
    if constexpr (G == 0)
        return k_test_select_flat<P>;
    else if constexpr (G == 1)
        return k_test_select_masked<P>;
    else
        return all ? k_test_select<G, P, true> : k_test_select<G, P, false>;
}

template <int G>
size_t construct_lds_bytes(int n) {
    return G == 1 ? masked_lds_bytes(n) : ant_lds_bytes(n);
}

template <int G, int P>
auto construct_kernel() {
    if constexpr (G == 0)
        return k_construct_flat<P>;
    else if constexpr (G == 1 || (G == 8 && P == 1))  // one pass: always with factors
        return k_construct_masked<P>;
    else
        return k_construct<G, P>;
}

// Calls f.template operator()<G, P>() for the tile and pass count of n, or
// with G = 0 and the number of 64-city blocks for rows of the flat layout, or
// with G = 1 and the pass count for tile 8 with the visited set as factors
// (`masked`).  Rows of five blocks at tile 8 take the factors: m = n = 320 0.119
// against 0.121 ms flat (converged 0.092 / 0.097), m = 65535 2.18 / 2.38.
template <typename F>
hipError_t dispatch_tile(int tile, int n, bool masked, F&& f) {
    static_assert(64 * kMaxFlatBlocks == kMaxFlatCities, "uses_lists");
    if (n <= (masked && tile == 8 ? kMaxOneLayoutCities : kMaxFlatCities)) return dispatch_flat(n, f);
    if (tile == 4) {
        switch ((n + 255) / 256) {
            case 2: return f.template operator()<4, 2>();
            case 3: return f.template operator()<4, 3>();
            case 4: return f.template operator()<4, 4>();
            default: return hipErrorInvalidValue;
        }
    }
    const int passes = (n + 511) / 512;
    if (masked) {
        switch (passes) {
            case 1: return f.template operator()<1, 1>();
            case 2: return f.template operator()<1, 2>();
            case 3: return f.template operator()<1, 3>();
            default: break;
        }
    }
    switch (passes) {
        case 1: return f.template operator()<8, 1>();
        case 2: return f.template operator()<8, 2>();
        case 3: return f.template operator()<8, 3>();
        case 4: return f.template operator()<8, 4>();
        case 5: return f.template operator()<8, 5>();
        case 6: return f.template operator()<8, 6>();
        case 7: return f.template operator()<8, 7>();
        case 8: return f.template operator()<8, 8>();
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool tile_supported(int tile, int n) {
    if (tile == 8) return n >= 1 && n <= kMaxCities;
    if (tile == 4) return n >= 1 && n <= 1024;
    return false;
}

const char* construct_layout(const Colony& c) {
    if (c.waves > 1) return "split";
    const char* name = "none";
    (void)dispatch_tile(c.tile, c.n, masked_rows(c.n, c.m), [&]<int G, int P>() {
        name = G == 0 ? "flat" : G == 1 ? "factors" : "bits";
        return hipSuccess;
    });
    return name;
}

int construct_occupancy(const Colony& c) {
    if (c.waves > 1) return construct_split_occupancy(c);
    int blocks = -1;
    (void)dispatch_tile(c.tile, c.n, masked_rows(c.n, c.m), [&]<int G, int P>() {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, construct_kernel<G, P>(), 64,
                                                         construct_lds_bytes<G>(c.n)) !=
            hipSuccess)
            blocks = -1;
        return hipSuccess;
    });
    return blocks;
}

hipError_t launch_construct(const Colony& c, uint32_t iter, hipStream_t s) {
    if (c.waves > 1) return launch_construct_split(c, iter, s);
    if (!tile_supported(c.tile, c.n)) return hipErrorInvalidValue;
    if (uses_lists(c)) {
        const hipError_t e = launch_short_lists(c, s);
        if (e != hipSuccess) return e;
    }
    return dispatch_tile(c.tile, c.n, masked_rows(c.n, c.m), [&]<int G, int P>() {
        hipLaunchKernelGGL((construct_kernel<G, P>()), dim3(c.m), dim3(64),
                           construct_lds_bytes<G>(c.n), s, c, iter);
        return hipGetLastError();
    });
}

hipError_t launch_construct_batch(const Colony* cols, const uint32_t* antmap, int total_ants,
                                  int max_n, size_t lds, hipStream_t s) {
    if (total_ants <= 0) return hipSuccess;
    if (max_n < 1 || max_n > kMaxCities) return hipErrorInvalidValue;
    const bool all = whole_rows_in_lds(total_ants);
    if (lds < (all ? batch_ants_lds_bytes<true>(max_n) : batch_ants_lds_bytes<false>(max_n)))
        return hipErrorInvalidValue;
    const int passes = (max_n + 511) / 512;
    const dim3 grid(total_ants), block(64);
    const auto launch = [&]<int P8>() {
        if (all)
            hipLaunchKernelGGL((k_construct_batch<P8, true>), grid, block, lds, s, cols, antmap);
        else
            hipLaunchKernelGGL((k_construct_batch<P8, false>), grid, block, lds, s, cols, antmap);
        return hipGetLastError();
    };
    if (passes <= 2) return launch.template operator()<2>();
    if (passes <= 4) return launch.template operator()<4>();
    if (passes <= 6) return launch.template operator()<6>();
    return launch.template operator()<8>();
}

hipError_t launch_test_select(int tile, bool batched, int n, int count, const float* rows,
                              const uint8_t* feasible, const float* u, int32_t* out,
                              hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (!tile_supported(tile, n)) return hipErrorInvalidValue;
    const int ld = (n + 63) & ~63;
    return dispatch_tile(tile, n, !batched, [&]<int G, int P>() {
        hipLaunchKernelGGL((test_select_kernel<G, P>(whole_rows_in_lds(count))), dim3(count), dim3(64), 0, s, rows, ld, n,
                           feasible, u, out);
        return hipGetLastError();
    });
}

}  // namespace aco
