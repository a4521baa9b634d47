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

// Lists of the n rows of colony c from its current choice matrix.
hipError_t launch_short_lists(const Colony& c, hipStream_t s);

}  // namespace aco
