// Counts of a bf16 row's values in LDS: sums over the whole vocabulary of any
// function of the logit from one pass over the row.
//
// A bf16 row has few distinct values: the weights of all its elements relative
// to a maximum that is only known once the row is read are sums of (count of a
// value) x (weight of the value).  Counting is one LDS add per element while
// the row streams; evaluating the weight of every element took a second pass
// of some 15 vector instructions per element and weight.  Streaming 512 rows
// of 128256 elements takes 21.6 us, with the counts 28.5 us.
//
// A table has one 32-bit word per magnitude from 2^-11 up to 2^9 (20 octaves
// of 128 values): positive values are counted in its low half, negative ones
// in its high half.  Larger magnitudes (-inf and row padding among them) are
// counted in 64 words past the magnitudes, one per lane, so that a masked row
// does not queue on one word; their values are not kept.  Smaller ones are
// counted in word 0: zeros (a padded vocabulary's columns, sparse logits), and
// others, which are listed with their values besides.  Counts that overflow
// a half change the table's total by 65,535 or 65,536 each and always
// downward, so the total shows whether any did.
//
// Lanes that meet on a word wait for each other, some five cycles each, so rows of
// few values (512 constant rows of 128256: 553 us a level, counted) are better
// not counted: four probes a batch tell how many lanes share a word with the
// first.  96 of 256 (a value that half of the row has) mark the list as full,
// which leaves the row to the caller's pass over its elements, and the batch is
// left out; at 48 a batch is left out if the list is full already.  (A quarter of
// the row at one value reaches 64 at most, and counting is the faster there:
// logits rounded to halves 80 us a level, by their elements 115.)  Eight probes
// cost a common row 2 % of its level.
#pragma once

#include "rheo_device.h"

namespace rheo {

constexpr uint32_t HIST_BASE = (116u << 7) - 1u;   // bf16 bits of 2^-11, less one
constexpr int HIST_MAGS = 20 * 128;                // magnitudes counted: words 1 .. HIST_MAGS
constexpr int HIST_OUT = HIST_MAGS + 1;            // first word of the larger magnitudes
constexpr int HIST_WORDS = HIST_OUT + WAVE;
constexpr int HIST_BYTES = 4 * HIST_WORDS;
constexpr int HIST_SMALL = 256;                    // values below 2^-11 and not 0 listed
static_assert(2 * HIST_BYTES <= 65536, "byte offsets of two tables in 16 bits");

typedef unsigned short hist_u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ hist_u16x2 hist_mags(uint32_t w) {
    return __builtin_bit_cast(hist_u16x2, w & 0x7FFF7FFFu);
}
// Whether a packed pair of bf16 holds a value below 2^-11 that is not 0.
__device__ __forceinline__ bool hist_has_small(hist_u16x2 least_less_1) {
    return least_less_1.x < HIST_BASE || least_less_1.y < HIST_BASE;
}
// The least of a vector's magnitudes, less 1 (0 wraps round to the largest).
__device__ __forceinline__ hist_u16x2 hist_least_less_1(const uint4& v) {
    const hist_u16x2 one = {1, 1};
    return __builtin_elementwise_min(
        __builtin_elementwise_min(hist_mags(v.x) - one, hist_mags(v.y) - one),
        __builtin_elementwise_min(hist_mags(v.z) - one, hist_mags(v.w) - one));
}

// Adds the vectors of a batch to a table.  `at` (the same in both halves):
// byte offset of the lane's table; small: the list's counter and entries
// (bf16 bits, `tag` in the upper half).
template <int NVB>
__device__ __forceinline__ void hist_add(uint8_t* tables, uint32_t at, const uint4 (&r)[NVB],
                                         int* small_n, uint32_t* small, uint32_t tag) {
    const uint32_t out = (uint32_t)(HIST_OUT + threadIdx.x % WAVE);
    const hist_u16x2 base = {(unsigned short)HIST_BASE, (unsigned short)HIST_BASE};
    const hist_u16x2 lim = {(unsigned short)out, (unsigned short)out};
    const hist_u16x2 four = {4, 4};
    const hist_u16x2 off = {(unsigned short)at, (unsigned short)at};
    int meet = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const hist_u16x2 i = __builtin_elementwise_min(
            __builtin_elementwise_sub_sat(hist_mags((&r[p * NVB / 2].x)[2 * p]), base), lim);
        const uint32_t lo = i.x, hi = i.y;
        meet += __popcll(__ballot(lo == lane_u32(lo, 0))) + __popcll(__ballot(hi == lane_u32(hi, 0)));
    }
    if (meet >= 3 * WAVE / 4) {
        if (meet >= 3 * WAVE / 2) {
            if (threadIdx.x % WAVE == 0) atomicAdd(small_n, HIST_SMALL + 1);
            return;
        }
        const int n = __hip_atomic_load(small_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_amdgcn_readfirstlane(n) > HIST_SMALL) return;
    }
#pragma unroll
    for (int e = 0; e < NVB; ++e) {
        const uint32_t* w = &r[e].x;
        hist_u16x2 least = {0xFFFF, 0xFFFF};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            hist_u16x2 i = __builtin_elementwise_sub_sat(hist_mags(w[c]), base);
            least = __builtin_elementwise_min(least, i);
            i = __builtin_elementwise_min(i, lim) * four + off;
            atomicAdd((uint32_t*)(tables + i.x), 1u << ((w[c] >> 11) & 16u));
            atomicAdd((uint32_t*)(tables + i.y), 1u << ((w[c] >> 27) & 16u));
        }
        if (__ballot(least.x == 0 || least.y == 0) != 0ull &&
            __ballot(hist_has_small(hist_least_less_1(r[e]))) != 0ull) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                for (int k = 0; k < 2; ++k) {
                    const uint32_t v = (w[c] >> (16 * k)) & 0xFFFFu;
                    if ((v & 0x7FFFu) - 1u < HIST_BASE) {
                        const int pos = atomicAdd(small_n, 1);
                        if (pos < HIST_SMALL) small[pos] = v | (tag << 16);
                    }
                }
            }
        }
    }
}

// The logit of magnitude word i (1 .. HIST_MAGS), positive.
__device__ __forceinline__ float hist_value(int i) {
    return __uint_as_float((HIST_BASE + (uint32_t)i) << 16);
}

}  // namespace rheo
