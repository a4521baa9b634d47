// shortlist.hpp -- the short list of every choice row: its largest entries,
// from which a selection over the whole row can often be made exactly.
//
// Both full-row rules (the roulette of Eq. (1) and the product rule of
// Section III-A) select from n cities, but a few entries carry nearly all of
// a row's weight once pheromone has gathered, and the product rule's winner
// is nearly always among the largest entries from the start.  Row i's list
// holds up to 63 of its largest entries in city order, with what bounds the
// rest of the row (the tail): the tail's weight before each entry, its whole
// weight and its largest entry.  A construction step reads the 512 bytes of
// the list first; where the bounds prove which city the rule over the whole
// row picks, that city is taken, else the whole row is read.  Either way the
// result is the rule's own, bit for bit; the list decides only what is read.
//
// Rows of more than 2560 cities have a wide list too, of up to 255 of the
// largest entries, four a lane: a step the short list does not settle tries
// it before the whole row, which for those rows comes from beyond the L2.
#pragma once

#include "aco_device.hpp"
#include "aco_state.hpp"

namespace aco {

constexpr int kListLanes = 64;                // list pitch: 63 entries, then the tail's entry
constexpr int kListEntries = kListLanes - 1;

// One entry: the weight's bits, and the city in the low 12 bits under the
// tail's weight before it, rounded up to 20 bits (an upper bound).  Lane 63
// holds the tail's largest entry and the tail's whole weight (+inf where the
// row must not be selected from by list).  Lanes past the entries: weight 0.
static_assert(kMaxCities <= 1 << 12, "a city takes 12 bits of an entry");

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// A wide list: the weights of entries 4 l .. 4 l + 3 at 16 l, their cities
// (uint16) at 1024 + 8 l, and at 1536 + 4 l the tail's weight before the last
// of them, an upper bound for all four.  Entry 255 is the tail's largest
// weight, lane 63's bound the tail's whole weight (+inf: not to be used).
// Past the entries: weight 0.
constexpr int kWideEntries = 255;
constexpr int kWideCities = 1024, kWideTails = 1536, kWideBytes = 1792;

struct WideEntries {
    float w[4];
    uint32_t cities[2];
    float tail;
    __device__ __forceinline__ int city(int e) const {
        return (int)((cities[e / 2] >> (16 * (e % 2))) & 0xFFFFu);
    }
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t wide_rsrc(const Colony& c) {
    return __builtin_amdgcn_make_buffer_rsrc(c.wide, (short)0, c.n * kWideBytes, 0x00020000);
}
__device__ __forceinline__ WideEntries load_wide(__amdgpu_buffer_rsrc_t wide, int row, int lane) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const int soff = row * kWideBytes;
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(wide, 16 * lane, soff, 0);
    const u32x2 c = __builtin_amdgcn_raw_buffer_load_b64(wide, kWideCities + 8 * lane, soff, 0);
    const uint32_t t = __builtin_amdgcn_raw_buffer_load_b32(wide, kWideTails + 4 * lane, soff, 0);
    WideEntries v;
    v.w[0] = __uint_as_float(w.x);
    v.w[1] = __uint_as_float(w.y);
    v.w[2] = __uint_as_float(w.z);
    v.w[3] = __uint_as_float(w.w);
    v.cities[0] = c.x;
    v.cities[1] = c.y;
    v.tail = __uint_as_float(t);
    return v;
}

__device__ __forceinline__ uint32_t list_meta(int city, float tail_above) {
    // tail_above >= +0; the next multiple of 2^11 in its bit pattern is not
    // below it (+inf stays +inf, 0 stays 0)
    const uint32_t b = __float_as_uint(tail_above);
    return (((b + 0x7FFu) >> 11) << 12) | (uint32_t)city;
}
__device__ __forceinline__ int list_city(uint32_t meta) { return (int)(meta & 0xFFFu); }
__device__ __forceinline__ float list_tail(uint32_t meta) {
    return __uint_as_float((meta >> 12) << 11);
}

// The lane's entry of the list of row `row`; lists: descriptor over the n
// rows.  The row goes in the scalar offset, so no vector address arithmetic
// sits between the selected city and the load.
__device__ __forceinline__ u32x2 load_list(__amdgpu_buffer_rsrc_t lists, int row, int lane) {
    return __builtin_amdgcn_raw_buffer_load_b64(lists, lane * (int)sizeof(u32x2),
                                                row * kListLanes * (int)sizeof(u32x2), 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t list_rsrc(const Colony& c) {
    return __builtin_amdgcn_make_buffer_rsrc(c.lists, (short)0,
                                             c.n * kListLanes * (int)sizeof(u32x2), 0x00020000);
}

// The roulette's selection from a row's short list alone (v: the lane's
// entry, w: its weight if its city is unvisited and the lane below 63, else 0,
// u: the step's draw): the bit of the chosen city's lane, or 0 where the step
// needs the whole row.
//
// The rule over the whole row picks the lowest unvisited city j whose prefix
// P_j exceeds target = fl32(u total).  With L_j the listed unvisited weight up
// to and including j, A_j the tail's weight before j and R its whole weight
// (both whether visited or not, so bounds from above), the exact sums obey
//   L_j <= prefix of j,  prefix of any city before j <= L_j - w_j + A_j,
//   L <= total <= L + R.
// So j is the rule's city if L_j > u (L + R) and L_j - w_j + A_j <= u L.  Every
// binary32 sum here and in the rule is a tree of non-negative terms of depth
// at most 13, and so within a factor (1 +- 2^-24)^13 of the exact one; the
// two sides of each test and their products together stay within 48 such
// factors, which the margin 1 +- 2^-18 (64 of them) covers.  (Sums are exact
// where they are subnormal; a list holds no weight below 2^-99, so L is 0,
// which passes no test, or keeps the products normal; and rows whose sums
// could pass 2^100 have R = +inf.)  Only one lane can pass both tests, and it
// is unvisited: with w_j = 0 they contradict each other.
__device__ __forceinline__ uint64_t roulette_list_hit(u32x2 v, float w, float u) {
    // u with the margin to either side, off the chain of the sums
    const float u_over = u * (1.0f + 0x1.0p-18f), u_under = u * (1.0f - 0x1.0p-18f);
    const float above = list_tail(v.y);
    const float s = s64_scan_in_place(w);
    const float listed = read_lane(s, 63), rest = read_lane(above, kListEntries);
    const float before = wave_shift_up1(s) + above;
    // two ballots and a scalar AND: the AND of the conditions would go
    // through a vector register
    return ballot(s > u_over * (listed + rest)) & ballot(before <= u_under * listed);
}

// The entry's weight where `unvisited` holds.
__device__ __forceinline__ float list_weight(u32x2 v, bool unvisited, int lane) {
    return ((lane < kListEntries) & unvisited) ? __uint_as_float(v.x) : 0.0f;
}

// The city of the lane that roulette_list_hit found.
__device__ __forceinline__ int hit_city(u32x2 v, uint64_t hit) {
    return list_city(__builtin_amdgcn_readlane(v.y, __builtin_ctzll(hit)));
}

// Whether the roulette tries the row's wide list: the city of entry 63.
__device__ __forceinline__ bool wide_tried(u32x2 v) {
    return list_city(__builtin_amdgcn_readlane(v.y, kListEntries)) != 0;
}

// The roulette's selection from a wide list, or -1: the tests of
// roulette_list_hit with four entries a lane (a sum is up to four additions
// deeper, so the sides of a test stay within 56 factors of the margin's 64).
// s_seen: city j's visited flag in byte j.
__device__ __forceinline__ int roulette_wide_pick(const WideEntries& v, const uint8_t* s_seen,
                                                  float u, int lane) {
    const float u_over = u * (1.0f + 0x1.0p-18f), u_under = u * (1.0f - 0x1.0p-18f);
    float w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool may = (4 * lane + e < kWideEntries) & (s_seen[v.city(e)] == 0);
        w[e] = may ? v.w[e] : 0.0f;
    }
    float in[4];  // prefixes inside the lane
    in[0] = w[0];
    in[1] = w[0] + w[1];
    in[2] = in[1] + w[2];
    in[3] = in[2] + w[3];
    const float s = s64_scan_in_place(in[3]);
    const float before = wave_shift_up1(s);
    const float listed = read_lane(s, 63), rest = read_lane(v.tail, 63);
    const float over = u_over * (listed + rest), under = u_under * listed;
    int j = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float prior = e ? before + in[e - 1] : before;
        const uint64_t hit = ballot(before + in[e] > over) & ballot(prior + v.tail <= under);
        if (hit) j = __builtin_amdgcn_readlane(v.city(e), __builtin_ctzll(hit));
    }
    return j;
}

// Whether the roulette of colony c may start its steps from the short lists
// (it then does where enough rows count, by_list): at tile 4 (n <= 256 by default)
// a step from the list takes longer than one from the row (n = 200: 0.41 against
// 0.37 us), except for the rows of five blocks that have the flat layout; and
// of up to 512 cities, up to 8 ants, one to an XCD's L2, gain nothing even
// when converged (n = 400, m = 8 0.150 against 0.146 ms; m = 16 0.127 against
// 0.150).  What builds the lists and what reads them ask this same question.
constexpr int kMinListCities = 256, kMaxFlatCities = 320;
__host__ __device__ inline bool uses_lists(const Colony& c) {
    return c.n > kMinListCities && (c.n <= kMaxFlatCities || c.tile == 8) && c.waves == 1 &&
           (c.n > 512 || c.m > 8);
}

// Bits of c.by_list[i]: whether row i counts for starting the steps of a
// construction from the lists (shortlist.hip).
constexpr uint32_t kRouletteRow = 1, kProductRow = 2;

// Whether half of colony c's rows count for the rule of bit `row_bit`; the same
// for every wavefront.
__device__ __forceinline__ bool half_by_list(const Colony& c, uint32_t row_bit, int lane) {
    const uint32_t mask = row_bit * 0x01010101u;
    int rows = 0;
    for (int j = 16 * lane; j < c.n; j += 16 * 64) {  // by_list is 0 past n
        const uint4 v = *reinterpret_cast<const uint4*>(c.by_list + j);
        rows += __popc(v.x & mask) + __popc(v.y & mask) + __popc(v.z & mask) + __popc(v.w & mask);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rows += __shfl_xor(rows, off);
    return 2 * __builtin_amdgcn_readfirstlane(rows) >= c.n;
}

// Lists of the n rows of colony c from its current choice matrix, and the
// rows that count for starting from them (c.by_list); wide lists where c.wide is
// not null.
hipError_t launch_short_lists(const Colony& c, hipStream_t s);
// As above for the first list_rows entries of a batch's rowmap ((colony << 16) |
// row, colony by colony); rows of colonies that use no lists are left out.
// max_n: the largest n among the colonies.
hipError_t launch_short_lists_batch(const Colony* cols, const uint32_t* rowmap, int list_rows,
                                    int max_n, hipStream_t s);
// The rows of `count` colonies (host), in their order, up to those of the last
// colony that uses lists.  Batches order colonies by falling n, so that the rest
// are those of the short rows, which use none.
int list_rows(const Colony* cols, int count);

}  // namespace aco
