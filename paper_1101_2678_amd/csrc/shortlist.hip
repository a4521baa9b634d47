// shortlist.hip -- builds the short list of every choice row (shortlist.hpp).
//
// One workgroup of four wavefronts per row; wavefront w takes the 64-city
// blocks w, w + 4, ...  A histogram over the top bits of the weights (eight
// bins an octave below the row's largest) gives the lowest bin edge that at
// most 63 entries reach; the entries above it go out in city order, each
// with the weight of all smaller ones before it.  Any subset of a row makes
// a correct list (what is left out is in the tail's bounds), so an edge
// between bins is as good as the exact 63 largest.
#include "shortlist.hpp"

namespace aco {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kBins = 256;
constexpr int kBinShift = 20;  // exponent and three bits of the significand
constexpr int kMaxBlocks = kMaxCities / 64;
// Sums of up to 4096 non-negative binary32 values by trees of depth at most
// 13 stay within a factor 1 +- 14 * 2^-24 of the exact sum.
constexpr float kUp = 1.0f + 0x1.0p-17f;
// Rows whose weights sum to this much are not selected from by list, so no
// sum or product of a step can overflow.
constexpr float kLargest = 0x1.0p100f;
// Weights below 2^-99 stay in the tail, so that the sums of a list's weights
// are 0 or far from underflow.
constexpr uint32_t kLeast = (127u - 99u) << 23;

// A row counts for starting the roulette's steps from the lists where the
// tail holds at most this share of it; a launch does so where half of the
// rows count.  A step the list does not settle reads the whole row after it,
// so the lists have to settle more than half of the steps unless the launch
// is bound by memory.  Shares at which lists and whole rows take the same time:
// n = 500 0.007, n = 1000 0.017, n = 1500 0.05 (0.02 with clustered cities), with
// m = n as with 256 ants.  Rows of four passes and more leave the L2, and the
// share follows what m ants ask for at once, 4 m n bytes: m n = 0.6e6 (n = 2400,
// m = 256) 0.06, 2.6e6 (1600, 1600) 0.04, 3e6 (3000, 1000) 0.10, 3.6e6 (1900, 1900)
// 0.18, 4.1e6 (4096, 1000) 0.31, 5.8e6 (2400, 2400) 0.55, 9e6 (3000, 3000) 0.6; n <
// 2000 and m of 4096 and 12000 0.2 to 0.28.  Lists from the first iteration where
// they settle little cost up to 48% (n = 2000, m = 256 2.32 against 1.56 ms; with
// beta = 1, n = 2400, m = 2400, 6.48 against 6.19).
__device__ __forceinline__ float by_list_share(int n, int m) {
    if (n <= 512) return 0.004f;
    if (n <= 1536) return 0.02f;
    const float x = 1e-6f * (float)m * (float)n;
    const float share = 0.001f * (x * x) * (x * x);
    const float most = n < 2000 ? 0.2f : 0.5f;
    return share < 0.02f ? 0.02f : share > most ? most : share;
}

// A row counts for the product rule's lists where the draws of its entries
// settle a step on the whole of a new tour with probability 1 - 2^-8 or more:
// entry j's product passes the tail's largest weight M unless r <= M / w_j, so
// that the entries together fail with probability prod M / w_j, and the sum
// of their log2(w_j / M) is at least an eighth of the bins between them and the
// first bin of the tail, summed over the entries.  With beta = 2 that sum is about
// 87 (w falls as 1 / j), with beta = 1 43; a launch starts from the lists where
// half of the rows count.  Without the vote, rows of equal weights (alpha = beta
// = 0, or beta = 0 on a new colony) paid for a list that settles nothing at
// every step: n = 100 0.053 -> 0.084 ms, 1000 0.86 -> 1.09, 2400 8.4 -> 9.7.
constexpr uint32_t kProductBins = 8 * 8;

// Wide lists: construction with m = n, without and with them, n = 3000 by
// iteration: 12.3 and 12.3 ms in the second (uniform cities), 2.10 and 2.16 in
// the 13th, 1.64 and 1.34 in the 24th; clustered cities 11.3 and 10.8, 1.95 and
// 1.86, 1.69 (20th) and 1.41.  Shorter rows gain the same in the end but lose
// on the way, where a whole row costs little more than the wide list that does
// not settle the step (n = 2400, 13th: 1.37 against 1.45; n = 2000: 0.92
// against 1.08).  The roulette tries the list of a row that leaves little to
// the tail: with 2% or 6% n = 3000 takes 122.1 and 122.8 ms for 24 iterations,
// clustered 20 in 89.0 and 87.9, with 0.1% 121.9 and 92.8, with all tried
// 135.6 and 89.1.
constexpr float kWideShare = 0.06f;

// One selection of a row's entries: those in the list, what is left of each
// block, and the largest left.
struct Selected {
    uint64_t mask[kMaxBlocks];
    float tail[kMaxBlocks];
    uint32_t tail_max[kWaves];
};

template <int TIERS>
struct ListShared {
    uint32_t bins[kBins];
    Selected tier[TIERS];
    float sum[kWaves];
    uint32_t max[kWaves];
};

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// The entries of tier `t` and what they leave, from the weights w of the
// wavefront's blocks.
template <int Q>
__device__ __forceinline__ void select_entries(const float (&w)[Q], uint32_t edge, uint32_t taken,
                                               int wave, int lane, Selected& t) {
    uint32_t tail_max = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = wave + kWaves * q;
        const uint32_t bits = __float_as_uint(w[q]);
        const bool in = bits >= kLeast && edge - (bits >> kBinShift) < taken;
        const uint64_t mask = ballot(in);
        tail_max = in || bits < tail_max ? tail_max : bits;
        const float s = s64_scan(in ? 0.0f : w[q]);
        if (lane == 63 && b < kMaxBlocks) {
            t.mask[b] = mask;
            t.tail[b] = s;
        }
    }
    tail_max = wave_max(tail_max);
    if (lane == 0) t.tail_max[wave] = tail_max;
}

// Calls out(rank, bits, city, tail before it) for every entry of the tier;
// returns their number, and the tail's weight in `rest`.
template <int Q, typename Out>
__device__ __forceinline__ int emit_entries(const float (&w)[Q], uint32_t edge, uint32_t taken,
                                            int blocks, int wave, int lane, const Selected& t,
                                            float& rest, Out&& out) {
    // block b's entries start at rank `first` of lane b, after a tail of
    // weight `weight` of lane b
    const uint32_t own = lane < blocks ? (uint32_t)__popcll(t.mask[lane]) : 0u;
    uint32_t first = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(first, off);
        first += lane >= off ? o : 0u;
    }
    const int entries = __builtin_amdgcn_readlane((int)first, 63);
    first -= own;
    const float weights = s64_scan(lane < blocks ? t.tail[lane] : 0.0f);
    const float weight = wave_shift_up1(weights);
    rest = read_lane(weights, 63) * kUp;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = wave + kWaves * q;
        if (b >= blocks) break;
        const uint32_t bits = __float_as_uint(w[q]);
        const bool in = bits >= kLeast && edge - (bits >> kBinShift) < taken;
        const uint64_t mask = ballot(in);
        if (mask == 0ull) continue;
        const float in_block = wave_shift_up1(s64_scan(in ? 0.0f : w[q]));
        const float above = (read_lane(weight, b) + in_block) * kUp;
        const int rank = __builtin_amdgcn_readlane((int)first, b) +
                         (int)__builtin_amdgcn_mbcnt_hi(
                             (uint32_t)(mask >> 32),
                             __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (in) out(rank, bits, 64 * b + lane, above, entries);
    }
    return entries;
}

__device__ __forceinline__ uint32_t max_of(const uint32_t (&v)[kWaves]) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) m = v[i] > m ? v[i] : m;
    return m;
}

// The lists of row i, with WIDE the wide one too: 256 threads, one pass over
// the row, held in registers.  Q: blocks of a wavefront,
// at least ceil(n / 256).
template <int Q, bool WIDE>
__device__ __forceinline__ void short_list_row(const Colony& c, int i,
                                               ListShared<WIDE ? 2 : 1>& sh) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = c.n;
    const float* row = c.choice + (size_t)i * c.ld;
    float w[Q];
    uint32_t top = 0;
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j = 64 * (wave + kWaves * q) + lane;
        w[q] = j < n ? row[j] : 0.0f;  // 0 on the diagonal
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        // weights are >= +0 and finite, so their bits order like the values
        // (a -0 restored by a caller shows as a bit pattern above all others)
        const uint32_t b = __float_as_uint(w[q]);
        top = b > top ? b : top;
        sum += w[q];
    }
    sh.bins[tid] = 0u;
    top = wave_max(top);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) {
        sh.max[wave] = top;
        sh.sum[wave] = sum;
    }
    __syncthreads();
    top = max_of(sh.max);
    const float total = (sh.sum[0] + sh.sum[1]) + (sh.sum[2] + sh.sum[3]);
    const uint32_t edge = top >> kBinShift;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t b = __float_as_uint(w[q]), bin = edge - (b >> kBinShift);
        if (b >= kLeast && bin < (uint32_t)kBins) atomicAdd(&sh.bins[bin], 1u);
    }
    __syncthreads();
    // bins 0 .. taken - 1 together hold at most 63 (wide: 255) entries
    uint32_t below = 0, cum[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) cum[e] = below += sh.bins[4 * lane + e];
    uint32_t before = below;  // inclusive scan over the lanes
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(before, off);
        before += lane >= off ? o : 0u;
    }
    before -= below;
    const auto bins_up_to = [&](uint32_t limit) {
        uint32_t bins = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) bins += before + cum[e] <= limit ? 1u : 0u;
        return (uint32_t)__builtin_amdgcn_readfirstlane(wave_sum(bins));
    };
    const uint32_t taken = bins_up_to(kListEntries);
    // sum over the entries of the bins from theirs to bin `taken`
    uint32_t above_tail = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        above_tail += 4u * (uint32_t)lane + (uint32_t)e < taken ? before + cum[e] : 0u;
    above_tail = wave_sum(above_tail);
    const uint32_t wide_taken = WIDE ? bins_up_to(kWideEntries) : 0u;
    select_entries<Q>(w, edge, taken, wave, lane, sh.tier[0]);
    if constexpr (WIDE) select_entries<Q>(w, edge, wide_taken, wave, lane, sh.tier[1]);
    __syncthreads();

    // not selected from by list: sums that could overflow, and weights that are
    // not finite or not above -0
    const bool bad = !(total < kLargest) || top >= 0x7F800000u;
    const float inf = __uint_as_float(0x7F800000u);
    const int blocks = (n + 63) >> 6;
    u32x2* out = reinterpret_cast<u32x2*>(c.lists) + (size_t)i * kListLanes;
    float rest;
    const int entries = emit_entries<Q>(
        w, edge, taken, blocks, wave, lane, sh.tier[0], rest,
        [&](int rank, uint32_t bits, int city, float above, int) {
            out[rank] = u32x2{bits, list_meta(city, above)};
        });
    if (tid == 0) {
        const bool roulette = entries > 0 && rest <= total * by_list_share(n, c.m);
        c.by_list[i] = (uint8_t)((roulette ? kRouletteRow : 0u) |
                                 (above_tail >= kProductBins ? kProductRow : 0u));
    }
    if (wave == 0 && lane >= entries && lane < kListEntries) out[lane] = u32x2{0u, 0u};
    const float short_rest = rest;
    int wide_tried = 0;
    if constexpr (WIDE) {
        uint8_t* base = c.wide + (size_t)i * kWideBytes;
        uint32_t* ww = reinterpret_cast<uint32_t*>(base);
        uint16_t* wc = reinterpret_cast<uint16_t*>(base + kWideCities);
        float* wt = reinterpret_cast<float*>(base + kWideTails);
        const int wide = emit_entries<Q>(
            w, edge, wide_taken, blocks, wave, lane, sh.tier[1], rest,
            [&](int rank, uint32_t bits, int city, float above, int count) {
                ww[rank] = bits;
                wc[rank] = (uint16_t)city;
                if (((rank & 3) == 3 || rank == count - 1) && rank < 4 * 63) wt[rank >> 2] = above;
            });
        // what no entry has written
        if (tid >= wide && tid < kWideEntries) {
            ww[tid] = 0u;
            wc[tid] = 0;
        }
        if (tid == kWideEntries) {
            ww[tid] = bad ? 0x7F800000u : max_of(sh.tier[1].tail_max);
            wc[tid] = 0;
        }
        if (tid < 64 && (4 * tid >= wide || tid == 63)) wt[tid] = bad ? inf : rest;
        wide_tried = rest <= total * kWideShare ? 1 : 0;
    }
    if (tid == kListEntries)
        out[kListEntries] = u32x2{bad ? 0x7F800000u : max_of(sh.tier[0].tail_max),
                                  list_meta(wide_tried, bad ? inf : short_rest)};
}

template <int Q, bool WIDE>
__global__ __launch_bounds__(kThreads) void k_short_lists(Colony c) {
    __shared__ ListShared<(WIDE ? 2 : 1)> sh;
    short_list_row<Q, WIDE>(c, blockIdx.x, sh);
}

// Rows of colonies that use no lists leave at once.  Rows of up to 512 cities
// have a body of their own in every launch: two blocks a wavefront.  Q > 10: some
// colonies have wide lists.
template <int Q>
__global__ __launch_bounds__(kThreads) void k_short_lists_batch(
    const Colony* __restrict__ cols, const uint32_t* __restrict__ rowmap) {
    __shared__ ListShared<1> sh;
    const uint32_t e = rowmap[blockIdx.x];
    const Colony c = cols[e >> 16];
    const int i = (int)(e & 0xffffu);
    if (!uses_lists(c)) return;
    if (c.n <= 512) {
        short_list_row<2, false>(c, i, sh);
        return;
    }
    if constexpr (Q > 10) {
        if (c.wide) {
            __shared__ ListShared<2> wide;
            short_list_row<Q, true>(c, i, wide);
            return;
        }
    }
    short_list_row<Q, false>(c, i, sh);
}

}  // namespace

hipError_t launch_short_lists_batch(const Colony* cols, const uint32_t* rowmap, int list_rows,
                                    int max_n, hipStream_t s) {
    if (list_rows <= 0) return hipSuccess;
    if (max_n < 1 || max_n > kMaxCities) return hipErrorInvalidValue;
    const dim3 grid(list_rows), block(kThreads);
    if (max_n <= 1024)
        hipLaunchKernelGGL(k_short_lists_batch<4>, grid, block, 0, s, cols, rowmap);
    else if (max_n <= 2560)
        hipLaunchKernelGGL(k_short_lists_batch<10>, grid, block, 0, s, cols, rowmap);
    else
        hipLaunchKernelGGL(k_short_lists_batch<16>, grid, block, 0, s, cols, rowmap);
    return hipGetLastError();
}

int list_rows(const Colony* cols, int count) {
    int rows = 0, upto = 0;
    for (int q = 0; q < count; ++q) {
        rows += cols[q].n;
        if (uses_lists(cols[q])) upto = rows;
    }
    return upto;
}

hipError_t launch_short_lists(const Colony& c, hipStream_t s) {
    if (c.n < 1 || c.n > kMaxCities) return hipErrorInvalidValue;
    const dim3 grid(c.n), block(kThreads);
    if (c.n <= 512)
        hipLaunchKernelGGL((k_short_lists<2, false>), grid, block, 0, s, c);
    else if (c.n <= 1024)
        hipLaunchKernelGGL((k_short_lists<4, false>), grid, block, 0, s, c);
    else if (c.n <= 2560)
        hipLaunchKernelGGL((k_short_lists<10, false>), grid, block, 0, s, c);
    else if (!c.wide)
        hipLaunchKernelGGL((k_short_lists<16, false>), grid, block, 0, s, c);
    else
        hipLaunchKernelGGL((k_short_lists<16, true>), grid, block, 0, s, c);
    static_assert(kMinWideCities == 2560, "the rows of k_short_lists<16>");
    return hipGetLastError();
}

}  // namespace aco
