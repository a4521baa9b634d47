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
// so where rows come from the L2 (n below about 2000) the lists have to
// settle more than half of the steps: at n = 1000 they do from the eighth
// iteration on (58% settled, 0.445 ms against 0.485 on whole rows; the first
// 0.81 against 0.48, the eleventh 0.331 against 0.48), when half of the rows
// leave 2% to the tail; rows of up to 512 cities, whose own step is shorter,
// two iterations later (n = 500: 0.168 against 0.184 ms in the ninth).  Longer
// rows are bound by memory, and the short reads leave room for the others
// from the first iteration (n = 2400: 5.9 against 6.1 ms, n = 2000 3.42 against
// 3.38 and from the second on less, n = 1800 3.00 against 2.37).
__device__ __forceinline__ float by_list_share(int n) {
    return n <= 512 ? 0.004f : n < 2000 ? 0.02f : 1.0f;
}

struct ListShared {
    uint32_t bins[kBins];
    uint64_t mask[kMaxBlocks];
    float tail[kMaxBlocks];
    float sum[kWaves];
    uint32_t max[kWaves], tail_max[kWaves];
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

// The list of row i.  Q: blocks of a wavefront, at least ceil(n / 256).
template <int Q>
__device__ __forceinline__ void short_list_row(const Colony& c, int i, ListShared& sh) {
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
#pragma unroll
    for (int v = 0; v < kWaves; ++v) top = sh.max[v] > top ? sh.max[v] : top;
    const float total = (sh.sum[0] + sh.sum[1]) + (sh.sum[2] + sh.sum[3]);
    const uint32_t edge = top >> kBinShift;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const uint32_t b = __float_as_uint(w[q]), bin = edge - (b >> kBinShift);
        if (b >= kLeast && bin < (uint32_t)kBins) atomicAdd(&sh.bins[bin], 1u);
    }
    __syncthreads();
    // bins 0 .. taken - 1 together hold at most 63 entries
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
    uint32_t taken = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) taken += before + cum[e] <= (uint32_t)kListEntries ? 1u : 0u;
    taken = __builtin_amdgcn_readfirstlane(wave_sum(taken));

    uint32_t tail_max = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = wave + kWaves * q;
        const uint32_t bits = __float_as_uint(w[q]);
        const bool in = bits >= kLeast && edge - (bits >> kBinShift) < taken;
        const uint64_t mask = ballot(in);
        const float t = in ? 0.0f : w[q];
        tail_max = in || bits < tail_max ? tail_max : bits;
        const float s = s64_scan(t);
        if (lane == 63 && b < kMaxBlocks) {
            sh.mask[b] = mask;
            sh.tail[b] = s;
        }
    }
    tail_max = wave_max(tail_max);
    if (lane == 0) sh.tail_max[wave] = tail_max;
    __syncthreads();
    // block b's entries start at rank `first` of lane b, after a tail of
    // weight `weight` of lane b
    const int blocks = (n + 63) >> 6;
    const uint32_t own = lane < blocks ? (uint32_t)__popcll(sh.mask[lane]) : 0u;
    uint32_t first = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(first, off);
        first += lane >= off ? o : 0u;
    }
    const int entries = __builtin_amdgcn_readlane((int)first, 63);
    first -= own;
    const float weights = s64_scan(lane < blocks ? sh.tail[lane] : 0.0f);
    const float weight = wave_shift_up1(weights);
    const float rest = read_lane(weights, 63) * kUp;

    u32x2* out = reinterpret_cast<u32x2*>(c.lists) + (size_t)i * kListLanes;
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
        if (in) out[rank] = u32x2{bits, list_meta(64 * b + lane, above)};
    }
    if (tid == 0) c.by_list[i] = entries > 0 && rest <= total * by_list_share(n) ? 1 : 0;
    if (wave == 0) {
        // not selected from by list: sums that could overflow, and weights
        // that are not finite or not above -0
        const bool bad = !(total < kLargest) || top >= 0x7F800000u;
        uint32_t m = 0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) m = sh.tail_max[v] > m ? sh.tail_max[v] : m;
        if (lane >= entries && lane < kListEntries) out[lane] = u32x2{0u, 0u};
        if (lane == kListEntries)
            out[lane] = u32x2{bad ? 0x7F800000u : m,
                              list_meta(0, bad ? __uint_as_float(0x7F800000u) : rest)};
    }
}

template <int Q>
__global__ __launch_bounds__(kThreads) void k_short_lists(Colony c) {
    __shared__ ListShared sh;
    short_list_row<Q>(c, blockIdx.x, sh);
}

template <int Q>
__global__ __launch_bounds__(kThreads) void k_short_lists_batch(
    const Colony* __restrict__ cols, const uint32_t* __restrict__ rowmap) {
    __shared__ ListShared sh;
    const uint32_t e = rowmap[blockIdx.x];
    const Colony c = cols[e >> 16];
    short_list_row<Q>(c, (int)(e & 0xffffu), sh);
}

}  // namespace

hipError_t launch_short_lists_batch(const Colony* cols, const uint32_t* rowmap, int total_rows,
                                    int max_n, hipStream_t s) {
    if (total_rows <= 0) return hipSuccess;
    if (max_n < 1 || max_n > kMaxCities) return hipErrorInvalidValue;
    const dim3 grid(total_rows), block(kThreads);
    if (max_n <= 1024)
        hipLaunchKernelGGL(k_short_lists_batch<4>, grid, block, 0, s, cols, rowmap);
    else if (max_n <= 2560)
        hipLaunchKernelGGL(k_short_lists_batch<10>, grid, block, 0, s, cols, rowmap);
    else
        hipLaunchKernelGGL(k_short_lists_batch<16>, grid, block, 0, s, cols, rowmap);
    return hipGetLastError();
}

hipError_t launch_short_lists(const Colony& c, hipStream_t s) {
    if (c.n < 1 || c.n > kMaxCities) return hipErrorInvalidValue;
    const dim3 grid(c.n), block(kThreads);
    if (c.n <= 1024)
        hipLaunchKernelGGL(k_short_lists<4>, grid, block, 0, s, c);
    else if (c.n <= 2560)
        hipLaunchKernelGGL(k_short_lists<10>, grid, block, 0, s, c);
    else
        hipLaunchKernelGGL(k_short_lists<16>, grid, block, 0, s, c);
    return hipGetLastError();
}

}  // namespace aco
