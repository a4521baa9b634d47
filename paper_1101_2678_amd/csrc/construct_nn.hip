// construct_nn.hip -- tour construction over nearest-neighbour candidate
// lists (Section II, the candidate-list variant of Eq. (1); the paper's GPU
// versions 4-6 of Table II).
//
// At city i the candidates are the entries of i's list (the nn nearest
// cities, ordered by (d_ij, j)).  If any of them is unvisited, the next city
// is drawn by the R64 roulette over the list in list order: lane r holds
// candidate r with weight choice[i][nnl[i][r]] if it is unvisited, else +0;
// one S64 prefix over the 64 lanes gives the prefixes, and the pick is the
// lowest unvisited r whose prefix exceeds fl32(u * total), else the highest
// unvisited r.  With a single 64-entry block the block offset is +0, so this
// is the full-row rule applied to the candidate vector.  If every candidate
// is visited, the next city is the unvisited city of largest choice value
// (lowest index among equal values), found by one pass over the row.
//
// One wavefront per ant.  Per step the wave reads one packed row of the
// candidate table (8 bytes per candidate, in L2 for every instance size the
// library accepts), so the kernel is bound by the latency of that dependent
// load and of the selection that follows it, not by bandwidth; the rare
// fallback takes the largest unvisited entry of the row's short list where
// rows are long, and otherwise, or where that holds none, issues all loads of
// the 4n-byte choice row at once.  The kernel
// is specialised on the number of 256-city passes of the fallback and on
// whether the list fits the low 32 lanes.
#include <hip/hip_runtime.h>

#include "aco_device.hpp"
#include "aco_state.hpp"
#include "nn.hpp"
#include "shortlist.hpp"

namespace aco {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

size_t round_up256(size_t v) { return (v + 255) & ~(size_t)255; }

__host__ __device__ size_t tour_bytes(int n) {
    return ((size_t)(n + 1) * sizeof(uint16_t) + 15) & ~(size_t)15;
}

// LDS of one ant: a visited flag per city (1 = visited, or >= n), then the
// tour.  Byte flags make a visit one plain byte store and let the fallback
// read the flags of four consecutive cities with one 32-bit load.
constexpr size_t kVisBytes = kMaxCities;

size_t construct_nn_lds(int n) { return kVisBytes + tour_bytes(n); }

// S64 restricted to lanes 0..31 (stage A and the row_bcast:15 step).  When
// lanes 32..63 hold +0, lanes 0..31 of the full tree end with these values
// and its last lane with the value of lane 31: row 3 adds (+0 + +0) + X
// with X = fl(R1 + R0), the value lane 31 gets here.
__device__ __forceinline__ float s64_scan_lo32(float x) {
    x = x + dpp_move<0x111, 0xF>(x);
    x = x + dpp_move<0x112, 0xF>(x);
    x = x + dpp_move<0x114, 0xF>(x);
    x = x + dpp_move<0x118, 0xF>(x);
    // in place, as in s64_scans
    asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf" : "+v"(x));
    return x;
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, kCtrl, kRowMask, 0xF, false);
}

// Wave maximum / minimum through the same DPP tree (lanes with no source
// take the neutral element); the result is read from lane 63, so it is
// wave-uniform.
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

// The unvisited city with the largest choice value, lowest index among equal
// values, for a row of n <= 256 P cities.  Choice values are finite and
// >= +0, so their bit patterns order like the values; key = bits + 1 (0 for
// "none").  Lane l holds cities 256 p + 4 l .. +3 of every pass p: all P
// loads are issued before any is used (loads past the row, rounded up to 4
// cities, return 0, and those cities are flagged visited).  Each lane keeps
// its first maximum in increasing city order; the wave takes the largest
// key, then the lowest city among the lanes holding it.
template <int P>
__device__ __forceinline__ int fallback_argmax(const float* row, int n, const uint8_t* vis,
                                               int lane) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(row), (short)0, ((n + 3) & ~3) * 4, 0x00020000);
    u32x4 q[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
        q[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, (256 * p + 4 * lane) * 4, 0, 0);
    uint32_t flags[P];
#pragma unroll
    for (int p = 0; p < P; ++p) flags[p] = reinterpret_cast<const uint32_t*>(vis)[64 * p + lane];
    // keep every load above in flight before the first use below (one memory
    // round trip instead of one per few passes)
    __builtin_amdgcn_sched_barrier(0);
    uint32_t best = 0;
    uint32_t best_j = ~0u;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t key = q[p][e] + 1u;
            if (((flags[p] >> (8 * e)) & 0xFFu) == 0u && key > best) {
                best = key;
                best_j = (uint32_t)(256 * p + 4 * lane + e);
            }
        }
    const uint32_t top = wave_max_u32(best);
    const uint32_t j = wave_min_u32(best == top && best != 0u ? best_j : ~0u);
    return top == 0u ? -1 : (int)j;
}

// The unvisited city with the largest choice value, from the row's short list,
// or -1 where the list holds none: it holds every city whose value is not
// below its smallest, in city order, so its largest unvisited value is the
// row's, on its lowest lane.
__device__ __forceinline__ int largest_listed(__amdgpu_buffer_rsrc_t lists, int row,
                                              const uint8_t* vis, int lane) {
    const u32x2 v = load_list(lists, row, lane);
    const int city = list_city(v.y);
    const bool may = (lane < kListEntries) & (vis[city] == 0);
    const uint32_t key = may ? v.x : 0u;
    const uint32_t top = wave_max_u32(key);
    // lane 63 holds +inf where the row must not be selected from by list
    const bool usable = (uint32_t)__builtin_amdgcn_readlane((int)v.x, kListEntries) < 0x7F800000u;
    if (top == 0u || !usable) return -1;
    return __builtin_amdgcn_readlane(city, __builtin_ctzll(ballot(key == top)));
}

// Packed candidate table from the current choice matrix.
__global__ __launch_bounds__(256) void k_cand_refresh(Colony c, NnTables t) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= c.n * t.kp) return;
    const int i = idx / t.kp, r = idx - i * t.kp;
    uint64_t v = 0;
    if (r < t.nn) {
        const int j = t.nnl[idx];
        v = ((uint64_t)j << 32) | __float_as_uint(c.choice[(size_t)i * c.ld + j]);
    }
    t.cand[idx] = v;
}

// Row i's list: the nn smallest of the keys (d_ij << 32) | j, in order.  Thread
// t holds the keys of cities t, t + 256, ...; the nn-th smallest of the 256
// threads' smallest keys bounds the nn-th smallest of all from above, so at
// most nn threads hold keys up to it, and the few keys up to it are ranked by
// counting the smaller ones.  Keys are distinct (j is); j = i and padding get
// the key 2^64 - 1 and are never taken because nn <= n - 1.  Three barriers
// instead of two for each entry: n = 100 26 -> 7.5 us, n = 1000 42 -> 15,
// n = 2400 84 -> 29 (nn = 32).
// Lists of up to four entries take a minimum of the workgroup an entry, which is
// shorter there (n = 1000, nn = 1 20 us a call against 28, n = 4096 33 against 55).
constexpr int kListThreads = 256;
constexpr int kMaxMinimumNn = 4;

struct NnShared {
    uint64_t least[kListThreads];
    uint64_t cand[kMaxNn * (kMaxCities / kListThreads)];
    uint64_t bound;
    uint32_t count;
};

// Of `count` keys in LDS, those smaller than `key`.
__device__ __forceinline__ int keys_below(const uint64_t* keys, int count, uint64_t key) {
    int r = 0;
    for (int i = 0; i < count; ++i) r += keys[i] < key ? 1 : 0;
    return r;
}

__device__ __forceinline__ void nn_list_row(const Colony& c, const NnTables& t, int i,
                                            NnShared& sh) {
    const int tid = threadIdx.x, n = c.n, nn = t.nn;
    uint64_t key[kMaxCities / kListThreads];
    uint64_t least = ~0ull;
#pragma unroll
    for (int q = 0; q < kMaxCities / kListThreads; ++q) {
        const int j = tid + kListThreads * q;
        key[q] = (j < n && j != i)
                     ? ((uint64_t)(uint32_t)c.dist[(size_t)i * c.ld + j] << 32) | (uint64_t)j
                     : ~0ull;
        least = key[q] < least ? key[q] : least;
    }
    uint16_t* out = t.nnl + (size_t)i * t.kp;
    for (int r = nn + tid; r < t.kp; r += kListThreads) out[r] = 0;
    if (nn <= kMaxMinimumNn) {
        for (int r = 0; r < nn; ++r) {
            uint64_t mn = least;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const uint64_t o = __shfl_xor((unsigned long long)mn, off);
                mn = o < mn ? o : mn;
            }
            // buffers by parity: one barrier an entry
            uint64_t* part = sh.least + 4 * (r & 1);
            if ((tid & 63) == 0) part[tid >> 6] = mn;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kListThreads / 64; ++w) mn = part[w] < mn ? part[w] : mn;
            if (tid == 0) out[r] = (uint16_t)(mn & 0xFFFFu);
            if (least == mn) {
                // this thread's smallest is taken: its next
                least = ~0ull;
#pragma unroll
                for (int q = 0; q < kMaxCities / kListThreads; ++q)
                    least = key[q] > mn && key[q] < least ? key[q] : least;
            }
        }
        return;
    }
    sh.least[tid] = least;
    if (tid == 0) sh.count = 0;
    __syncthreads();
    if (least != ~0ull && keys_below(sh.least, kListThreads, least) == nn - 1) sh.bound = least;
    __syncthreads();
    const uint64_t bound = sh.bound;
#pragma unroll
    for (int q = 0; q < kMaxCities / kListThreads; ++q)
        if (key[q] <= bound) sh.cand[atomicAdd(&sh.count, 1u)] = key[q];
    __syncthreads();
    const int count = (int)sh.count;
    for (int q = tid; q < count; q += kListThreads) {
        const uint64_t k = sh.cand[q];
        const int r = keys_below(sh.cand, count, k);
        if (r < nn) out[r] = (uint16_t)(k & 0xFFFFu);
    }
}

__global__ __launch_bounds__(kListThreads) void k_nn_lists(Colony c, NnTables t) {
    __shared__ NnShared sh;
    nn_list_row(c, t, blockIdx.x, sh);
}

// The initialisation's lists of colony c: up to 32 entries a row, in the
// successor table (n x mp uint16, mp >= 64), which is not used before the
// first construction.
__host__ __device__ NnTables init_tables(const Colony& c) {
    NnTables t{};
    t.nn = c.n - 1 < 32 ? c.n - 1 : 32;
    t.kp = 32;
    t.nnl = c.succ;
    t.cand = nullptr;
    return t;
}

__global__ __launch_bounds__(kListThreads) void k_nn_lists_batch(
    const Colony* __restrict__ cols, const uint32_t* __restrict__ rowmap) {
    __shared__ NnShared sh;
    const uint32_t e = rowmap[blockIdx.x];
    const Colony c = cols[e >> 16];
    nn_list_row(c, init_tables(c), (int)(e & 0xffffu), sh);
}

// Rows of more than 1280 cities have their short lists built: a step that
// leaves its candidate list (2% of them) then reads 512 bytes instead of 4n.
// With the launch for the lists, construction with nn = 30, mean of 20
// iterations: n = 3000 1.26 -> 1.13 ms, n = 2400 0.836 -> 0.790, n = 1500
// 0.442 -> 0.439, n = 1000 0.265 both, n = 100 0.0346 -> 0.0390.
// Fewer than 64 ants leave too few such steps for the launch (n = 1300 with 4
// ants 0.483 -> 0.504 ms, n = 2400 with 64 0.663 -> 0.657), and without the heuristic
// (beta = 0) a new colony's rows have no list (n = 2400, m = n 0.919 -> 0.978 ms).
// What builds the lists and what reads them ask nn_uses_lists.
constexpr int kMinNnListPasses = 6;
constexpr int kMinNnListAnts = 64;
__host__ __device__ inline bool nn_uses_lists(const Colony& c) {
    return c.n > 256 * (kMinNnListPasses - 1) && c.m >= kMinNnListAnts && c.beta > 0;
}
template <int P>
constexpr bool kNnLists = P >= kMinNnListPasses;

template <int P, bool kNn32>
__global__ __launch_bounds__(64) void k_construct_nn(Colony c, NnTables t, uint32_t iter) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint8_t* s_vis = smem;
    uint16_t* s_tour = reinterpret_cast<uint16_t*>(smem + kVisBytes);
    const int lane = threadIdx.x;
    const int k = ant_of_block(blockIdx.x, c.m);
    const int n = c.n, nn = t.nn, kp = t.kp;
    const PhiloxKey key{(uint32_t)c.seed, (uint32_t)(c.seed >> 32)};

    for (int w = lane; w < (int)(kVisBytes / 4); w += 64) {
        uint32_t f = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) f |= (4 * w + b >= n ? 1u : 0u) << (8 * b);
        reinterpret_cast<uint32_t*>(s_vis)[w] = f;
    }
    __syncthreads();

    const uint32_t x0 = draw(key, iter, (uint32_t)k, 0u);
    int cur = (int)(((uint64_t)x0 * (uint64_t)(uint32_t)n) >> 32);

    // Lanes kp..63 re-read entries of the same row (kp is 32 or 64), so the
    // load needs no branch; only lanes < nn can be candidates.
    const int col = lane & (kp - 1);
    const bool in_list = lane < nn;
    const uint64_t list_mask = nn == 64 ? ~0ull : (1ull << nn) - 1ull;
    // the row offset goes in the scalar offset, so no vector address math sits
    // between the selected city and the next load (every access is in range)
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(
        t.cand, (short)0, n * kp * (int)sizeof(uint64_t), 0x00020000);
    const __amdgpu_buffer_rsrc_t lists = list_rsrc(c);
    const bool use_lists = kNnLists<P> && nn_uses_lists(c);
    // A step's candidate row is loaded as soon as its city is known; the
    // city's bookkeeping (tour entry, visited flag) follows the load, before
    // the flags are read (one wavefront: its LDS accesses stay in order).  64
    // steps at a time, with their draws.
    for (int base = 0; base < n - 1; base += 64) {
        const float u64 = uniform24(draw(key, iter, (uint32_t)k, (uint32_t)(base + 1 + lane)));
        const int count = __builtin_amdgcn_readfirstlane(n - 1 - base < 64 ? n - 1 - base : 64);
        int i = 0;
        do {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(
                crs, col * (int)sizeof(uint64_t), cur * kp * (int)sizeof(uint64_t), 0);
            if (lane == 0) {
                s_tour[base + i] = (uint16_t)cur;
                s_vis[cur] = 1;
            }
            const float u = read_lane(u64, i);
            const int city = (int)v.y;
            // every lane reads its flag (a valid index on every lane), so the
            // read needs no branch; `&` keeps it unconditional
            const bool unvisited = s_vis[city] == 0;
            const bool feas = in_list & unvisited;
            const float w = feas ? __uint_as_float(v.x) : 0.0f;
            const float s = kNn32 ? s64_scan_lo32(w) : s64_scan_in_place(w);
            // opaque, or the product becomes a scalar read, a move and a product
            float goal = u * s;
            asm("" : "+v"(goal));
            const float target = read_lane(goal, kNn32 ? 31 : 63);
            const uint64_t live = ballot(unvisited) & list_mask;
            int next;
            if (__builtin_expect(live != 0, 1)) {
                const uint64_t hit = ballot(s > target) & live;
                const int r = hit ? __builtin_ctzll(hit) : 63 - __builtin_clzll(live);
                next = __builtin_amdgcn_readlane(city, r);
            } else {
                next = use_lists ? largest_listed(lists, cur, s_vis, lane) : -1;
                if (next < 0) {
                    next = fallback_argmax<P>(c.choice + (size_t)cur * c.ld, n, s_vis, lane);
                    // at least one city is unvisited, so next >= 0; the clamp
                    // only keeps the LDS indices in range should that ever
                    // break.
                    next = next < 0 ? 0 : next;
                }
            }
            cur = __builtin_amdgcn_readfirstlane(next);
        } while (++i < count);
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

// Launches k_construct_nn<P, nn <= 32> for P = ceil(n / 256) in 1..16.
template <int P>
hipError_t launch_nn_passes(const Colony& c, const NnTables& t, uint32_t iter, hipStream_t s) {
    if constexpr (P > kMaxCities / 256) {
        return hipErrorInvalidValue;
    } else {
        if ((c.n + 255) / 256 != P) return launch_nn_passes<P + 1>(c, t, iter, s);
        const size_t lds = construct_nn_lds(c.n);
        if (t.nn <= 32)
            hipLaunchKernelGGL((k_construct_nn<P, true>), dim3(c.m), dim3(64), lds, s, c, t, iter);
        else
            hipLaunchKernelGGL((k_construct_nn<P, false>), dim3(c.m), dim3(64), lds, s, c, t,
                               iter);
        return hipGetLastError();
    }
}

// The unseen city nearest to the row's city (smallest d, lowest index among
// equal d), for a row of n <= 256 P cities: all P 16-byte loads are issued
// before any is used; loads past the row (rounded up to 4 cities) return 0,
// and those cities are flagged seen.  -1 if every city is seen.
template <int P>
__device__ __forceinline__ int nearest_unseen(const int32_t* row, int n, const uint8_t* seen,
                                              int lane) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(row), (short)0, ((n + 3) & ~3) * 4, 0x00020000);
    u32x4 q[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
        q[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, (256 * p + 4 * lane) * 4, 0, 0);
    uint32_t flags[P];
#pragma unroll
    for (int p = 0; p < P; ++p) flags[p] = reinterpret_cast<const uint32_t*>(seen)[64 * p + lane];
    __builtin_amdgcn_sched_barrier(0);
    uint32_t best = ~0u, best_j = ~0u;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // distances are >= 1 and < 2^31, so ~0 never stands for a city
            const uint32_t d = ((flags[p] >> (8 * e)) & 0xFFu) ? ~0u : q[p][e];
            if (d < best) {
                best = d;
                best_j = (uint32_t)(256 * p + 4 * lane + e);
            }
        }
    const uint32_t top = wave_min_u32(best);
    const uint32_t j = wave_min_u32(best == top ? best_j : ~0u);
    return top == ~0u ? -1 : (int)j;
}

// C_nn, the length of the nearest-neighbour tour from city 0 (ties to the
// lowest index), and tau0 = fl32(m / C_nn).  Row i of the (d, j)-sorted lists
// holds i's nearest cities, so its first unseen entry is the nearest unseen
// city overall (every city off the list has a larger (d, j) key); only when
// every entry is seen does the wave scan the whole distance row.  One
// wavefront walks; the tour is kept in LDS and summed at the end.  A step is
// a chain of dependent reads, so the workgroup first copies the first `staged`
// entries of every list to LDS (32 where they fit, to n = 2350, else 16;
// n = 100 28 -> 18 us, n = 1000 290 -> 159, n = 2400 712 -> 400).  That takes up
// to a compute unit's whole LDS.  Beside other work (the server's admissions)
// rows of more than 512 cities stage nothing: a workgroup of more than 40 KB then
// waits until enough ants on some compute unit have ended.  Mean and longest
// walk in a trace of requests, staged / not: n <= 256 0.04, 0.07 / 0.09, 0.22 ms;
// n <= 512 0.07, 0.10 / 0.19, 0.86; n <= 1024 0.45, 6.3 / 0.50, 2.2; n <= 1536 3.1,
// 10.3 / 0.73, 1.6; n <= 2048 0.90, 4.6 / 0.89, 2.3.
constexpr int kMaxStagedBeside = 512;
constexpr int kTourThreads = 256;
constexpr size_t kTourLds = 160u << 10;

__host__ __device__ size_t nn_tour_lds(int n, int staged) {
    return kVisBytes + tour_bytes(n) + (size_t)n * staged * sizeof(uint16_t);
}
__host__ __device__ int staged_entries(int n) { return nn_tour_lds(n, 32) <= kTourLds ? 32 : 16; }

template <int P, bool STAGED>
__device__ __forceinline__ void nn_tour(const Colony& c, const NnTables& t, unsigned char* smem) {
    const int n = c.n, nn = t.nn, kp = t.kp, staged = STAGED ? staged_entries(n) : kp;
    uint8_t* s_seen = smem;
    uint16_t* s_tour = reinterpret_cast<uint16_t*>(smem + kVisBytes);
    uint16_t* s_list = reinterpret_cast<uint16_t*>(smem + kVisBytes + tour_bytes(n));
    const int tid = threadIdx.x;
    for (int w = tid; w < (int)(kVisBytes / 4); w += kTourThreads) {
        uint32_t f = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) f |= (4 * w + b >= n || 4 * w + b == 0 ? 1u : 0u) << (8 * b);
        reinterpret_cast<uint32_t*>(s_seen)[w] = f;
    }
    if (tid == 0) s_tour[0] = 0;
    // 16-byte pieces of eight entries; kp = 32
    const int pieces = staged / 8;
    for (int q = tid; STAGED && q < n * pieces; q += kTourThreads) {
        const int i = q / pieces, e = q - i * pieces;
        reinterpret_cast<uint4*>(s_list)[q] =
            *reinterpret_cast<const uint4*>(t.nnl + (size_t)i * kp + 8 * e);
    }
    __syncthreads();
    if (tid >= 64) return;  // no barrier follows
    const int lane = tid;
    const int held = staged < nn ? staged : nn;
    const bool in_held = lane < held;
    const int col = lane & (staged - 1);
    int cur = 0;
    for (int step = 1; step < n; ++step) {
        const int city = STAGED ? s_list[cur * staged + col] : t.nnl[(size_t)cur * kp + col];
        uint64_t live = ballot(in_held & (s_seen[city] == 0));
        int next;
        if (__builtin_expect(live != 0ull, 1)) {
            next = __builtin_amdgcn_readlane(city, __builtin_ctzll(live));
        } else {
            // the entries past the staged ones, then the whole row
            int more = 0;
            if (STAGED) {
                more = t.nnl[(size_t)cur * kp + (lane & 31)];
                live = ballot((lane < nn) & (s_seen[more] == 0));
            }
            if (live) {
                next = __builtin_amdgcn_readlane(more, __builtin_ctzll(live));
            } else {
                next = nearest_unseen<P>(c.dist + (size_t)cur * c.ld, n, s_seen, lane);
                // n - step >= 1 cities are unseen, so next >= 0; the clamp only
                // keeps the LDS indices in range should that ever break.
                next = next < 0 ? 0 : next;
            }
        }
        next = __builtin_amdgcn_readfirstlane(next);
        if (lane == 0) {
            s_tour[step] = (uint16_t)next;
            s_seen[next] = 1;
        }
        cur = next;
    }
    long long len = 0;
    for (int s = lane; s < n; s += 64) {
        const int i = s_tour[s], j = s + 1 < n ? s_tour[s + 1] : 0;
        len += c.dist[(size_t)i * c.ld + j];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) len += __shfl_xor(len, off);
    if (lane == 0) {
        *c.cnn = len;
        *c.tau0 = (float)((double)c.m / (double)len);
        *c.best_len = 0x7fffffffffffffffLL;
    }
}

template <int P, bool STAGED>
__global__ __launch_bounds__(kTourThreads) void k_nn_tour(Colony c) {
    extern __shared__ __align__(16) unsigned char smem[];
    nn_tour<P, STAGED>(c, init_tables(c), smem);
}

// Workgroup q: the tour of colony cols[q]; every colony has n <= 256 P.
template <int P>
__global__ __launch_bounds__(kTourThreads) void k_nn_tour_batch(const Colony* __restrict__ cols) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Colony c = cols[blockIdx.x];
    nn_tour<P, true>(c, init_tables(c), smem);
}

// Calls f.template operator()<P>() for a P of 1, 2, 4, 6, 8, 10, 12 or 16 with
// n <= 256 P: a row scan's passes beyond n read nothing.
template <typename F>
hipError_t dispatch_scan_passes(int n, F&& f) {
    const int p = (n + 255) / 256;
    if (p <= 1) return f.template operator()<1>();
    if (p <= 2) return f.template operator()<2>();
    if (p <= 4) return f.template operator()<4>();
    if (p <= 6) return f.template operator()<6>();
    if (p <= 8) return f.template operator()<8>();
    if (p <= 10) return f.template operator()<10>();
    if (p <= 12) return f.template operator()<12>();
    return f.template operator()<kMaxCities / 256>();
}

}  // namespace

hipError_t launch_nn_tour(const Colony& c, bool alone, hipStream_t s) {
    if (c.n < 2 || c.n > kMaxCities || c.mp < 32) return hipErrorInvalidValue;
    hipError_t e = launch_nn_lists(c, init_tables(c), s);
    if (e != hipSuccess) return e;
    return dispatch_scan_passes(c.n, [&]<int P>() {
        if (alone || c.n <= kMaxStagedBeside)
            hipLaunchKernelGGL((k_nn_tour<P, true>), dim3(1), dim3(kTourThreads),
                               nn_tour_lds(c.n, staged_entries(c.n)), s, c);
        else
            hipLaunchKernelGGL((k_nn_tour<P, false>), dim3(1), dim3(kTourThreads),
                               nn_tour_lds(c.n, 0), s, c);
        return hipGetLastError();
    });
}

hipError_t launch_nn_tour_batch(const Colony* cols, const Colony* host_cols, int count,
                                const uint32_t* rowmap, int total_rows, int max_n,
                                hipStream_t s) {
    if (count <= 0 || total_rows <= 0) return hipSuccess;
    if (max_n < 2 || max_n > kMaxCities) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_nn_lists_batch, dim3(total_rows), dim3(kListThreads), 0, s, cols, rowmap);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // every colony's request: a smaller one may stage more entries a row
    size_t lds = 0;
    for (int q = 0; q < count; ++q) {
        const int n = host_cols[q].n;
        if (n < 2 || n > max_n) return hipErrorInvalidValue;
        const size_t need = nn_tour_lds(n, staged_entries(n));
        lds = need > lds ? need : lds;
    }
    return dispatch_scan_passes(max_n, [&]<int P>() {
        hipLaunchKernelGGL(k_nn_tour_batch<P>, dim3(count), dim3(kTourThreads), lds, s, cols);
        return hipGetLastError();
    });
}

size_t nn_table_bytes(int n, int nn) {
    const size_t kp = (size_t)nn_pitch(nn);
    return round_up256((size_t)n * kp * sizeof(uint16_t)) +
           round_up256((size_t)n * kp * sizeof(uint64_t));
}

NnTables nn_carve(char* base, int n, int nn) {
    NnTables t{};
    t.nn = nn;
    t.kp = nn_pitch(nn);
    t.nnl = reinterpret_cast<uint16_t*>(base);
    t.cand = reinterpret_cast<uint64_t*>(base +
                                         round_up256((size_t)n * t.kp * sizeof(uint16_t)));
    return t;
}

hipError_t launch_nn_lists(const Colony& c, const NnTables& t, hipStream_t s) {
    if (t.nn < 1 || t.nn > kMaxNn || t.nn > c.n - 1 || c.n > kMaxCities)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_nn_lists, dim3(c.n), dim3(kListThreads), 0, s, c, t);
    return hipGetLastError();
}

hipError_t launch_construct_nn(const Colony& c, const NnTables& t, uint32_t iter, hipStream_t s) {
    if (t.nn < 1 || t.nn > kMaxNn || t.nn > c.n - 1 || c.n > kMaxCities)
        return hipErrorInvalidValue;
    const int cells = c.n * t.kp;
    hipLaunchKernelGGL(k_cand_refresh, dim3((cells + 255) / 256), dim3(256), 0, s, c, t);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && nn_uses_lists(c)) {
        Colony short_only = c;
        short_only.wide = nullptr;
        e = launch_short_lists(short_only, s);
    }
    if (e != hipSuccess) return e;
    return launch_nn_passes<1>(c, t, iter, s);
}

}  // namespace aco
