// What the row kernels share: reading a logit row, streaming it through a
// block while its largest elements are found, and the sorted top of the row.
#pragma once

#include <type_traits>

#include "code_hist.h"
#include "rheo_device.h"
#include "rheo_state.h"
#include "pool_common.h"

namespace rheo {

constexpr int SMAX = 1024;    // largest support
constexpr int NTE = 512;      // threads per k_expand_row block
constexpr int EBATCH = 8;     // 16-byte vectors per thread and batch of k_expand_row
constexpr int kLargeSupport = 256;  // supports above it: the large class of k_expand_row

template <int DT>
__device__ __forceinline__ float elem(const uint4& v, int k) {
    const uint32_t* w = &v.x;
    if (DT) return (k & 1) ? bf_hi(w[k >> 1]) : bf_lo(w[k >> 1]);
    return __uint_as_float(w[k]);
}

// Vector vi (VEC consecutive elements) of a row; elements past V read as
// bf16 0xFFFF (a NaN: it drops out of the raw-word maxima below, whose
// kernels run with the IEEE mode bit clear, and its order code 0 lies below
// that of -inf) or fp32 -inf (ranked after every logit by its id).  Every
// consumer also checks the index against V.
template <int DT>
__device__ __forceinline__ uint4 load_row_vec(const char* base, int vi, int V) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int ESZ = DT ? 2 : 4;
    const int e = vi * VEC;
    if (e + VEC <= V) return load_stream16(base + (int64_t)e * ESZ);
    uint32_t w[4];
    if (DT) {
        const uint16_t* p16 = (const uint16_t*)base;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e0 = e + 2 * q;
            const uint32_t lo = (e0 < V) ? p16[e0] : 0xFFFFu;
            const uint32_t hi = (e0 + 1 < V) ? p16[e0 + 1] : 0xFFFFu;
            w[q] = lo | (hi << 16);
        }
    } else {
        const uint32_t* p32 = (const uint32_t*)base;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (e + q < V) ? p32[e + q] : 0xFF800000u;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// LDS layout of the pool kernel's dynamic buffer: the chunk lists and one
// empty list after them, the support, ranking keys and per-entry
// arrays; the level's priority keys (256 of them) reuse the regions of the
// support and the ranking keys.
struct PoolLds {
    int m, top, k2, w1, q, wr, xs, bytes;
};
__host__ __device__ inline int pad16(int x) { return (x + 15) & ~15; }
__host__ __device__ inline PoolLds pool_lds(int S, int C) {
    PoolLds L;
    const int S2 = S > 256 ? S : 256;
    L.m = 0;
    L.top = L.m + pad16(8 * (C + 1) * S);
    L.k2 = L.top + pad16(8 * S2);
    L.w1 = L.k2 + pad16(8 * S2);
    L.q = L.w1 + pad16(4 * S);
    L.wr = L.q + pad16(4 * S);
    L.xs = L.wr + pad16(2 * S);
    L.bytes = L.xs + pad16(2 * S);
    return L;
}

// The parent of row j of sequence b: frontier node j of the previous level
// (the n_expand children with the highest priority, chosen by the previous
// launch), with the Philox draw of its sampled slot (keyed by that launch's
// rng_key and the parent's uid).  One thread.  The load is issued by
// row_parent_load, the draw may be taken early (has_u), and row_parent
// checks both, so a kernel can do this work while it streams its row.
struct RowParentRaw {
    int pu;
    uint64_t u;
};
__device__ __forceinline__ RowParentRaw row_parent_load(const TreeDev& t, const LevelArgs& a,
                                                        int b, int j) {
    RowParentRaw r{0, 0ull};
    if (a.level > 0) r.pu = t.frontier[(int64_t)b * t.NE + j];
    return r;
}
__device__ __forceinline__ uint64_t parent_draw(const LevelArgs& a, int b, int pu) {
    return philox_draw(a.fr_key, P_DRAFT, (uint64_t)b, (uint64_t)pu);
}
__device__ __forceinline__ void row_parent(const TreeDev& t, const LevelArgs& a, int b, int j,
                                           const RowParentRaw& raw, bool has_u, int* s_pu,
                                           uint64_t* s_u) {
    const int level = a.level, K = t.K, NE = t.NE;
    int pu = raw.pu;
    const int lo_uid = (level == 0) ? 0 : ((level == 1) ? 1 : 1 + K + (level - 2) * NE * K);
    const int hi_uid = (level == 0) ? 1 : lo_uid + ((level == 1) ? 1 : NE) * K;
    if (pu < lo_uid || pu >= hi_uid) {
        atomicOr(t.err, 16);
        pu = 0;
    }
    *s_pu = pu;
    // the root (level 0, or the fallback above) is drawn with this launch's key
    *s_u = (pu == 0) ? philox_draw(a.rng_key, P_DRAFT, (uint64_t)b, 0ull)
                     : (has_u ? raw.u : parent_draw(a, b, pu));
}

// max(a, b, c) in one instruction; with the IEEE mode bit clear (the
// caller's kernel runs ieee_mode_off first) a NaN operand is ignored.
// Volatile: kept in program order after the mode change.
__device__ __forceinline__ float max3_nan_drop(float a, float b, float c) {
    float r;
    asm volatile("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Exact maximum element of a vector of eight bf16 (raw word bits: a packed
// word read as fp32 is its high element plus a fraction of one bf16 ulp made
// of the low element's bits, so the maximum over the raw words and the
// unpacked low elements, with its low 16 bits cleared, is exactly the
// largest element).  A word whose high element is -inf (and low element not
// +0) is a NaN and is dropped, which loses nothing: -inf is the least
// logit, and the low element counts through its own unpacked operand.
// Padding (0xFFFF) drops out the same way; a vector of padding alone gives
// a NaN (order code 0).  Returned with garbage in the low 16 bits.
__device__ __forceinline__ uint32_t bf16x8_max_raw(const uint4& v) {
    float m = max3_nan_drop(__uint_as_float(v.x), bf_lo(v.x), __uint_as_float(v.y));
    m = max3_nan_drop(m, bf_lo(v.y), __uint_as_float(v.z));
    m = max3_nan_drop(m, bf_lo(v.z), __uint_as_float(v.w));
    m = max3_nan_drop(m, bf_lo(v.w), bf_lo(v.w));
    return __float_as_uint(m);
}

typedef short rs_short2 __attribute__((ext_vector_type(2)));
typedef unsigned short rs_ushort2 __attribute__((ext_vector_type(2)));
// Order codes of two packed bf16 values (negative: all bits flipped,
// otherwise the sign bit set), two lanes of 16 bits at once.
__device__ __forceinline__ rs_ushort2 bf16x2_codes(uint32_t w) {
    const rs_short2 s = __builtin_bit_cast(rs_short2, w);
    const uint32_t m = __builtin_bit_cast(uint32_t, (rs_short2)(s >> (short)15)) | 0x80008000u;
    return __builtin_bit_cast(rs_ushort2, w ^ m);
}

// Lane l (a constant) of v replaced by the wave-uniform s.
__device__ __forceinline__ int writelane_i32(int v, int s, int l) {
    asm volatile("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(s), "n"(l));
    return v;
}

// h = the largest 16-bit code that at least nsel of the offered codes reach
// (c1 and c2 of every thread, and c3 and c4 too if `four`, a block-uniform
// flag), four bits per round: each wave counts its offers >= h | d << sh
// for d = 1..15 with ballots, lane d of the wave stores that count, the
// waves' counts are added, and d is the largest one whose count still
// reaches nsel.  s_cnt holds 2 * (NT / WAVE) * 16 ints.  Needs nsel <= the
// number of offers; all threads of the block call it.
template <int NT>
__device__ __forceinline__ uint32_t offer_threshold(uint32_t c1, uint32_t c2, uint32_t c3,
                                                    uint32_t c4, bool four, int nsel,
                                                    int* s_cnt) {
    constexpr int NW = NT / WAVE;
    const int lane = threadIdx.x % WAVE, wid = threadIdx.x / WAVE;
    uint32_t h = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int sh = 12 - 4 * r;
        int* buf = s_cnt + (r & 1) * NW * 16;
        // h has no bits at or below this digit, so c >= h | d << sh is
        // ((c - h, saturated at 0) >> sh) >= d: a compare with a small constant
        const uint32_t e1 = __builtin_elementwise_sub_sat(c1, h) >> sh;
        const uint32_t e2 = __builtin_elementwise_sub_sat(c2, h) >> sh;
        const uint32_t e3 = __builtin_elementwise_sub_sat(c3, h) >> sh;
        const uint32_t e4 = __builtin_elementwise_sub_sat(c4, h) >> sh;
        int mine = 0;
        if (four) {
#pragma unroll
            for (int d = 1; d < 16; ++d) {
                const uint32_t cd = (uint32_t)d;
                const int n = __popcll(__ballot(e1 >= cd)) + __popcll(__ballot(e2 >= cd)) +
                              __popcll(__ballot(e3 >= cd)) + __popcll(__ballot(e4 >= cd));
                mine = writelane_i32(mine, n, d);
            }
        } else {
#pragma unroll
            for (int d = 1; d < 16; ++d) {
                const uint32_t cd = (uint32_t)d;
                const int n = __popcll(__ballot(e1 >= cd)) + __popcll(__ballot(e2 >= cd));
                mine = writelane_i32(mine, n, d);
            }
        }
        if (lane < 16) buf[wid * 16 + lane] = mine;
        __syncthreads();
        int tot = 0;
        if (lane < 16) {
#pragma unroll
            for (int w = 0; w < NW; ++w) tot += buf[w * 16 + lane];
        }
        const uint64_t ok = __ballot(lane >= 1 && lane < 16 && tot >= nsel);
        const uint32_t d = ok ? (uint32_t)(63 - __builtin_clzll(ok)) : 0u;
        h |= d << sh;
    }
    return h;
}
template <int NT>
__device__ __forceinline__ uint32_t offer_threshold(uint32_t c1, uint32_t c2, int nsel,
                                                    int* s_cnt) {
    return offer_threshold<NT>(c1, c2, 0u, 0u, false, nsel, s_cnt);
}

// Adds 1 to s_hist[d] for every lane with `in`: one add for all the lanes that share
// the first such lane's digit, so that equal elements do not queue on a word.
__device__ __forceinline__ void count_digit(int* s_hist, uint32_t d, bool in) {
    const uint64_t all = __ballot(in);
    if (all == 0ull) return;
    const int lead = (int)__builtin_ctzll(all);
    const uint64_t same = __ballot(in && d == lane_u32(d, lead));
    const int lane = threadIdx.x % WAVE;
    if (lane == lead) atomicAdd(&s_hist[d], __popcll(same));
    else if (in && !((same >> lane) & 1ull)) atomicAdd(&s_hist[d], 1);
}

// Exact selection for a degenerate range: more candidates than LDS holds
// (massive ties at the threshold, large values crowded into few threads, or a
// support near the number of the row's vectors, whose maxima then bound
// nothing).  The range is NQ vectors per thread, vector q of this thread at
// index vfirst + q * NT + tid; elements at V and beyond do not count;
// push(v, id) records an element.  It re-reads the range, four vectors at a
// time, once per pass.
//
// bf16: count the elements whose code lies above the threshold code h, and those
// at it; if the nsel-th largest element has code h, x = h; if it lies above h
// and the elements above h fit (at most cap), take those.  Otherwise, and for fp32, x
// = the nsel-th largest code (bf16: the 16-bit order code, fp32: the 32-bit
// one) by its digits from the top, 8 bits a pass, each from a histogram of
// the elements that share the digits before.  Then everything above x and the
// smallest ids among those at x (ranks of the ties in id order from per-wave
// counts and wave scans), until `taken` says that nsel are pushed.  By bisection of the 64-bit key, in 64 passes, a level of
// 1000 bf16 elements at support 128 took 197 us, of 2500 fp32 elements at
// support 1024 180; so they take 33 and 53.
//
// s_scr holds max(256, NQ * NT / WAVE) ints.  Ends with a barrier.
template <int DT, int NT, int NQ, typename Push>
__device__ void exact_select_fallback(const char* base, int V, int vfirst, uint32_t h, int nsel,
                                      int cap, Push push, int* taken, int* s_redi, int* s_scr) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int NW = NT / WAVE;
    static_assert(NQ % 4 == 0 && NQ <= 64, "re-read in groups of four vectors");
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    int (*s_tie)[NW] = (int (*)[NW])s_scr;
    // the vectors of the range inside the row, in groups of four; the opaque trip
    // count keeps each pass a loop (re-reading per pass) rather than one
    // straight-line block holding every element
    int nq = __builtin_amdgcn_readfirstlane(
        min(NQ, (((V + VEC - 1) / VEC - vfirst + NT - 1) / NT + 3) & ~3));
    asm volatile("" : "+s"(nq));
    auto group = [&](int q0, uint4 (&w)[4]) {
        // an opaque index keeps every pass's loads (and what is computed
        // from them) inside its loop instead of live across the passes
        int vf = vfirst;
        asm volatile("" : "+v"(vf));
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = load_row_vec<DT>(base, vf + (q0 + q) * NT + tid, V);
    };
    auto code = [](float v) { return DT ? ord32(v) >> 16 : ord32(v); };
    // (past the row bf16 elements read as code 0, below every x; fp32 ones as -inf)
    auto inside = [&](int e) { return DT || e < V; };
    // elements at x in every vector, per wave; and those above it, in all
    auto count_ties = [&](uint32_t x) {
        int ngt = 0;
#pragma unroll 1
        for (int q0 = 0; q0 < nq; q0 += 4) {
            uint4 w[4];
            group(q0, w);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e0 = (vfirst + (q0 + q) * NT + tid) * VEC;
                int nt = 0;
#pragma unroll
                for (int k = 0; k < VEC; ++k) {
                    const uint32_t c = code(elem<DT>(w[q], k));
                    ngt += (int)(inside(e0 + k) && c > x);
                    nt += (int)(inside(e0 + k) && c == x);
                }
                const int tot = wave_sum_i32(nt);
                if (lane == 0) s_tie[q0 + q][wid] = tot;
            }
        }
        return block_sum_i32<NT>(ngt, s_redi);
    };
    uint32_t x = h;                              // the nsel-th largest code
    int need = 0;                                // elements to take at it
    bool found = false;
    if (DT) {
        x = max(h, 1u);
        const int ngt = count_ties(x);
        need = nsel - ngt;
        found = need > 0;
        if (!found && ngt <= cap) {
            need = 0;                            // (all above h, none at it)
            nsel = ngt;
            found = true;
        }
    }
    if (!found) {
        x = 0;
        need = nsel;
#pragma unroll 1
        for (int sh = DT ? 8 : 24; sh >= 0; sh -= 8) {
            __syncthreads();                     // (the digit before is read)
            for (int i = tid; i < 256; i += NT) s_scr[i] = 0;
            __syncthreads();
#pragma unroll 1
            for (int q0 = 0; q0 < nq; q0 += 4) {
                uint4 w[4];
                group(q0, w);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int e0 = (vfirst + (q0 + q) * NT + tid) * VEC;
#pragma unroll
                    for (int k = 0; k < VEC; ++k) {
                        const uint32_t c = code(elem<DT>(w[q], k));
                        count_digit(s_scr, (c >> sh) & 255u,
                                    (DT ? c != 0u : e0 + k < V) && ((c ^ x) >> sh) >> 8 == 0u);
                    }
                }
            }
            __syncthreads();
            // every wave finds the largest digit that `need` elements reach; lane l
            // holds digits 4 l .. 4 l + 3
            int cnt[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                cnt[k] = s_scr[4 * lane + k];
                sum += cnt[k];
            }
            const int ex = wave_excl_scan(sum);
            int above = (int)lane_u32((uint32_t)(ex + sum), WAVE - 1) - ex - sum;
            int digit = -1, left = 0;
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                if (above < need && above + cnt[k] >= need) {
                    digit = 4 * lane + k;
                    left = need - above;
                }
                above += cnt[k];
            }
            const uint64_t own = __ballot(digit >= 0);     // one lane: nsel <= the range
            const int l = own ? (int)__builtin_ctzll(own) : 0;
            x |= lane_u32((uint32_t)max(digit, 0), l) << sh;
            need = (int)lane_u32((uint32_t)left, l);
        }
        __syncthreads();
        (void)count_ties(x);
    }
    __syncthreads();
    // ties at x are taken in id order: vector q, then thread, then element
    int prior = 0;                               // ties in the vectors before q, all threads
#pragma unroll 1
    for (int q0 = 0; q0 < nq; q0 += 4) {
        const int n = __hip_atomic_load(taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_amdgcn_readfirstlane(n) >= nsel) break;
        uint4 w[4];
        group(q0, w);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e0 = (vfirst + (q0 + q) * NT + tid) * VEC;
            int rk = 0;
            if (need > 0) {
                int nt = 0;
#pragma unroll
                for (int k = 0; k < VEC; ++k)
                    nt += (int)(inside(e0 + k) && code(elem<DT>(w[q], k)) == x);
                rk = prior + wave_excl_scan(nt);
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) {
                    rk += (ww < wid) ? s_tie[q0 + q][ww] : 0;
                    prior += s_tie[q0 + q][ww];
                }
            }
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                const float v = elem<DT>(w[q], k);
                const uint32_t cd = code(v);
                if (inside(e0 + k)) {
                    if (cd > x) {
                        push(v, e0 + k);
                    } else if (cd == x) {
                        if (rk < need) push(v, e0 + k);
                        ++rk;
                    }
                }
            }
        }
    }
    __syncthreads();
}

// The candidate count after exact_select_fallback (which ends with a
// barrier): an atomic load behind a compiler barrier, since the call is not
// inlined and a plain load of the counter may be scheduled before it.
__device__ __forceinline__ int fallback_count(int* cnt) {
    asm volatile("" ::: "memory");
    return __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Dynamic LDS of a row kernel's block (160 KB less the static): the limit set
// for each of them, the same whatever tree sets it, since it belongs to the
// kernel and every tree launches under it.
constexpr size_t kRowLdsMax = 156 * 1024;

constexpr int NBINS = 512;    // histogram bins of the ranking (LS: twice as many)
constexpr int ROW_BATCHES = 8;  // most batches of a row: 64 vectors per thread

// LDS of k_expand_row: the vector codes, which the ranked candidates and the
// pool's ranking keys replace once the candidates are gathered; the
// candidates; the histogram and the bins' starts (before them, the waves'
// candidate-vector lists); the arrays the pool is formed from.
struct RowLds {
    PoolLds p;                 // p.k2: also the ranked candidates, over the codes
    int codes, keys, hist, start;
    int tab, small;            // counts of the row's values (bf16)
};
// How a row kernel counts its row's values: not at all; in two tables by the
// lane's parity (fewer lanes meet on one word); in one table per batch.
enum Count { COUNT_NONE = 0, COUNT_ROW = 1, COUNT_BATCH = 2 };
// Candidates a block holds: about 1.4 of the selected in common rows.
__host__ __device__ constexpr int row_cap(bool ls, int count) {
    return ls ? 2048 : count == COUNT_BATCH ? 512 : 960;
}
__host__ __device__ inline RowLds row_lds(int S, bool ls, int nb, int ntb, int count) {
    RowLds L;
    const int cap = row_cap(ls, count), nbins = ls ? 2 * NBINS : NBINS;
    const int S2 = S > 256 ? S : 256;
    int o = (count == COUNT_BATCH ? 8 : 16) * ntb * nb;     // codes
    if (o < 8 * cap) o = 8 * cap;
    L.codes = 0;
    L.p.m = 0;
    L.p.k2 = 0;
    L.keys = o;
    o += 8 * cap;
    L.hist = o;
    o += 4 * nbins;
    L.start = o;
    const int lists = 4 * (ntb / WAVE) * WAVE * (ls ? 2 : 1);
    o += lists > 4 * nbins ? lists : 4 * nbins;
    L.p.top = o;
    o += pad16(8 * S2);
    L.p.w1 = o;
    o += pad16(4 * S);
    L.p.q = o;
    o += pad16(4 * S);
    L.p.wr = o;
    o += pad16(2 * S);
    L.p.xs = o;
    o += pad16(2 * S);
    L.tab = o;
    if (count) o += pad16((count == COUNT_BATCH && nb > 2 ? nb : 2) * HIST_BYTES);
    L.small = o;
    if (count) o += 4 * HIST_SMALL;
    L.p.bytes = o;
    return L;
}

// The largest of the four 16-bit code offers over the wave.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    x = max(x, row_ror<8>(x));
    x = max(x, row_ror<4>(x));
    x = max(x, row_ror<2>(x));
    x = max(x, row_ror<1>(x));
    return max(max(lane_u32(x, 0), lane_u32(x, 16)), max(lane_u32(x, 32), lane_u32(x, 48)));
}

// A 16-bit code that at least k of the wave's offers reach (two per lane, or
// four), the largest one with its two lowest bits clear (a sixteenth of an
// octave at most below the k-th largest offer): two bits a round, whose three
// counts do not wait for each other.
template <bool FOUR>
__device__ __forceinline__ uint32_t wave_kth_code(uint32_t c1, uint32_t c2, uint32_t c3,
                                                  uint32_t c4, int k) {
    uint32_t h = 0;
    auto reach = [&](uint32_t x) -> bool {
        int n = __popcll(__ballot(c1 >= x)) + __popcll(__ballot(c2 >= x));
        if (FOUR) n += __popcll(__ballot(c3 >= x)) + __popcll(__ballot(c4 >= x));
        return n >= k;
    };
#pragma unroll
    for (int sh = 14; sh >= 2; sh -= 2) {
        const bool r1 = reach(h | (1u << sh)), r2 = reach(h | (2u << sh)), r3 = reach(h | (3u << sh));
        h |= (uint32_t)((int)r1 + (int)r2 + (int)r3) << sh;
    }
    return h;
}

// The largest code that S of the row's vector codes reach, at most NBIN - 1 above
// h, which S of them reach (returned where fewer do: codes of two vectors).
// s_hist holds zeros, and does again; *s_at is any word.  All threads of the block
// call it.
template <int NTB, int NBIN>
__device__ __forceinline__ uint32_t codes_threshold(const uint32_t* codes, int words, uint32_t h,
                                                    int S, int* s_hist, int* s_red, int* s_at) {
    constexpr int BPT = NBIN > NTB ? NBIN / NTB : 1;
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    if (tid == 0) *s_at = 0;
#pragma unroll 1
    for (int i = tid; i < words; i += NTB) {
        const uint32_t w = codes[i], lo = w & 0xFFFFu, hi = w >> 16;
        if (lo >= h) atomicAdd(&s_hist[min(lo - h, (uint32_t)(NBIN - 1))], 1);
        if (hi >= h) atomicAdd(&s_hist[min(hi - h, (uint32_t)(NBIN - 1))], 1);
    }
    __syncthreads();
    const int top_bin = NBIN - 1 - tid * BPT;
    int hv[BPT], tot = 0;
#pragma unroll
    for (int r = 0; r < BPT; ++r) {
        hv[r] = top_bin - r >= 0 ? s_hist[top_bin - r] : 0;
        tot += hv[r];
    }
    int st = wave_excl_scan(tot);
    if (lane == WAVE - 1) s_red[wid] = st + tot;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NTB / WAVE; ++w) st += (w < wid) ? s_red[w] : 0;
#pragma unroll
    for (int r = 0; r < BPT; ++r) {
        if (st < S && st + hv[r] >= S) *s_at = top_bin - r;
        st += hv[r];
        if (top_bin - r >= 0) s_hist[top_bin - r] = 0;
    }
    __syncthreads();
    return h + (uint32_t)*s_at;
}

// The maximum of a vector, exact in its high 16 bits (fp32: truncated).
template <int DT>
__device__ __forceinline__ uint32_t vec_max_raw(const uint4& v) {
    if (DT) return bf16x8_max_raw(v);
    return __float_as_uint(fmaxf(fmaxf(__uint_as_float(v.x), __uint_as_float(v.y)),
                                 fmaxf(__uint_as_float(v.z), __uint_as_float(v.w))));
}

// Shared state of a row kernel's block.
template <int NTB>
struct RowShared {
    int thr[2 * (NTB / WAVE) * 16];
    int wcode[NTB / WAVE], red[NTB / WAVE];
    int cnt, nsmall, pu;
    uint64_t u;
};

// Whether a level's rows are read with ordinary loads: those of a few rows stay
// in the L2s (4 MB on each of 8 XCDs) for the second read of the candidates
// (8 rows of 128256 bf16: 16.6 us a level with streaming loads, 15.5 with
// these); those of many evict each other (512 rows: 33.6 against 34.7 us).
inline bool level_cached(const TreeDev& t, int rows) {
    return (int64_t)rows * t.stride * (t.dtype ? 2 : 4) <= (16 << 20);
}

// A row as a block of NTB threads reads it: vector q of a thread is lane
// `lane` of the 64-vector slot (wave + q) mod waves of block stride q; a batch
// is EBATCH strides.  Rotating the slot spreads every wave's reads over all
// offsets of a stride; with a fixed slot per wave the waves of a block
// finished streaming up to several µs apart.
template <int DT, int NTB>
struct RowReader {
    const char* base;
    int V, NVF, wsu, lane;
    bool cached;               // the level's rows stay in the L2s (see level_cached)
    __device__ __forceinline__ int vidx(int q) const {
        return (((wsu + q) & (NTB / WAVE - 1)) * WAVE + lane) + NTB * q;
    }
    __device__ __forceinline__ void load_batch(uint4 (&r)[EBATCH], int bt) const {
        // plain loads where every lane of the block reads whole vectors
        if (NTB * (bt * EBATCH + EBATCH) <= NVF) {
            if (cached) {
#pragma unroll
                for (int e = 0; e < EBATCH; ++e)
                    r[e] = *(const uint4*)(base + (int64_t)vidx(bt * EBATCH + e) * 16);
            } else {
#pragma unroll
                for (int e = 0; e < EBATCH; ++e)
                    r[e] = load_stream16(base + (int64_t)vidx(bt * EBATCH + e) * 16);
            }
        } else {
#pragma unroll
            for (int e = 0; e < EBATCH; ++e) {
                const int q = bt * EBATCH + e;
                if (NTB * (q + 1) <= NVF) r[e] = load_stream16(base + (int64_t)vidx(q) * 16);
                else r[e] = load_row_vec<DT>(base, vidx(q), V);
            }
        }
    }
};
template <int DT, int NTB>
__device__ __forceinline__ RowReader<DT, NTB> row_reader(const TreeDev& t, const LevelArgs& a,
                                                         int row) {
    RowReader<DT, NTB> rd;
    rd.base = (const char*)a.logits + (int64_t)row * t.stride * (DT ? 2 : 4);
    rd.V = t.V;
    rd.NVF = t.V / (DT ? 8 : 4);
    rd.wsu = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    rd.lane = threadIdx.x % WAVE;
    rd.cached = a.cached != 0;
    return rd;
}
template <int DT, int NTB>
__host__ __device__ __forceinline__ int row_batches(int V) {
    constexpr int PER = NTB * EBATCH * (DT ? 8 : 4);
    return (V + PER - 1) / PER;
}

// ---------------------------------------------------------------------------
// row_top: streams the row, and leaves its S largest elements by (logit desc,
// id asc) in s_top (LDS, sorted).  Also takes the row's parent and its draw
// (rs.pu, rs.u) and, on request, counts the row's values (code_hist.h).
// Returns the parent's record and the row maximum (fp32: truncated).
//
// The row is streamed once, in double-buffered batches of EBATCH 16-byte
// vectors per thread; of every vector only its exact maximum is kept, as a
// 16-bit order code in LDS (one 16-byte store per thread and batch).  Each
// wave then takes the ceil(S / waves)-th largest of the maxima its lanes
// offer, and the least of the waves' values is a threshold that at least S
// elements reach: one block barrier.  Every wave reads its own candidate
// vectors again and appends their elements at or above the threshold to the
// block's candidates (about 1.4 S of them), which are ranked by a
// histogram: bins linear in the value, their starts from one prefix sum,
// and the order inside a bin by counting.
//
// What bounds it: the stream, then the latency of the steps after it (HBM is
// idle while a row that has no successor on its compute unit ranks).
// COUNT_BATCH keeps one code for two vectors (it selects few elements, and its
// tables need the LDS).
// ---------------------------------------------------------------------------
struct RowTop {
    ParentRec pr;
    float vmax;
};
template <int DT, bool LS, int NTB, int CNT>
__device__ __forceinline__ RowTop row_top(const TreeDev& t, const LevelArgs& a, int row, int S,
                                          uint8_t* lds, const RowLds& L,
                                          const RowReader<DT, NTB>& rd, RowShared<NTB>& rs) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int NW = NTB / WAVE;
    constexpr int CC = row_cap(LS, CNT);        // candidates held
    constexpr int NBIN = LS ? 2 * NBINS : NBINS;
    constexpr int BPT = NBIN > NTB ? NBIN / NTB : 1;   // bins per thread
    constexpr int KPT = (CC + NTB - 1) / NTB;   // candidates per thread
    constexpr int RND = LS ? 2 : 1;             // candidate vectors per lane and round
    constexpr bool PAIR = CNT == COUNT_BATCH;   // one code per two vectors
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int b = row / a.P, j = row % a.P;
    const int K = t.K, V = t.V;
    const int level = a.level;
    const int NB = row_batches<DT, NTB>(V);
    uint64_t* s_keys = (uint64_t*)(lds + L.keys);
    uint64_t* s_ord = (uint64_t*)(lds + L.p.k2);
    uint64_t* s_top = (uint64_t*)(lds + L.p.top);
    int* s_hist = (int*)(lds + L.hist);
    int* s_start = (int*)(lds + L.start);
    uint8_t* s_tab = lds + L.tab;
    uint32_t* s_small = (uint32_t*)(lds + L.small);

    // the parent's frontier entry is loaded while the row streams (after its
    // first loads are issued when there are several batches), its draw taken
    // while the last batches are in flight, and both checked after the row is
    // streamed
    RowParentRaw rp{0, 0ull};
    bool has_u = false;
    if (tid == 0) rs.cnt = 0;
    for (int i = tid; i < S; i += NTB) s_top[i] = 0ull;   // id -1 until ranked
    for (int i = tid; i < NBIN; i += NTB) s_hist[i] = 0;
    if (CNT) {
        const int words = (CNT == COUNT_BATCH && NB > 2 ? NB : 2) * HIST_WORDS;
        for (int i = tid; i < words; i += NTB) ((uint32_t*)s_tab)[i] = 0;
        if (tid == 0) rs.nsmall = 0;
    }

    // ---- the row, streamed ---------------------------------------------------
    // p1, p2: the two largest codes of the even (low half) and of the odd
    // vectors
    rs_ushort2 p1 = {0, 0}, p2 = {0, 0};
    auto proc_batch = [&](const uint4 (&r)[EBATCH], int bt) {
        uint32_t cw[EBATCH / 2];
#pragma unroll
        for (int e = 0; e < EBATCH; e += 2) {
            const uint32_t lo = vec_max_raw<DT>(r[e]), hi = vec_max_raw<DT>(r[e + 1]);
            rs_ushort2 cq = bf16x2_codes(__builtin_amdgcn_perm(hi, lo, 0x07060302u));
            // fp32 vectors past the row hold -inf: code 0 instead, as bf16 ones have,
            // or short rows would list thousands of them as candidates (400 to 900
            // elements at support 128: 29 us a level against 16)
            if (DT == 0 && NTB * (bt + 1) * EBATCH > rd.NVF) {
                const int q = bt * EBATCH + e;
                if (rd.vidx(q) * VEC >= V) cq.x = 0;
                if (rd.vidx(q + 1) * VEC >= V) cq.y = 0;
            }
            cw[e / 2] = __builtin_bit_cast(uint32_t, cq);
            if (LS) p2 = __builtin_elementwise_max(p2, __builtin_elementwise_min(p1, cq));
            p1 = __builtin_elementwise_max(p1, cq);
        }
        if (CNT == COUNT_ROW)
            hist_add(s_tab, (uint32_t)(lane & 1) * HIST_BYTES, r, &rs.nsmall, s_small, 0u);
        if (CNT == COUNT_BATCH)
            hist_add(s_tab + bt * HIST_BYTES, 0u, r, &rs.nsmall, s_small, (uint32_t)bt);
        if (PAIR) {
            // vectors e and e + 2 of every four share a code
            uint32_t pw[2];
#pragma unroll
            for (int e = 0; e < 2; ++e)
                pw[e] = __builtin_bit_cast(
                    uint32_t, __builtin_elementwise_max(
                                  __builtin_bit_cast(rs_ushort2, cw[2 * e]),
                                  __builtin_bit_cast(rs_ushort2, cw[2 * e + 1])));
            ((uint2*)(lds + L.codes))[bt * NTB + tid] = make_uint2(pw[0], pw[1]);
        } else {
            ((uint4*)(lds + L.codes))[bt * NTB + tid] = make_uint4(cw[0], cw[1], cw[2], cw[3]);
        }
    };
    static_assert(EBATCH == 8, "the codes of a batch in one store");
    if (NB <= 2 && tid == 0) rp = row_parent_load(t, a, b, j);
    if (CNT) __syncthreads();                    // (the tables are clear)
    {
        uint4 ra[EBATCH], rb[EBATCH];
        rd.load_batch(ra, 0);
        for (int bt = 0; bt < NB; bt += 2) {
            if (bt + 1 < NB) rd.load_batch(rb, bt + 1);
            proc_batch(ra, bt);
            if (bt + 2 < NB) rd.load_batch(ra, bt + 2);
            if (NB > 2 && bt == 0 && tid == 0) rp = row_parent_load(t, a, b, j);
            // the parent's draw (a serial Philox chain) while the last batch is
            // in flight, once the parent's load has returned
            if (bt + 2 >= NB && tid == 0 && level > 0) {
                rp.u = parent_draw(a, b, rp.pu);
                has_u = true;
            }
            if (bt + 1 < NB) proc_batch(rb, bt + 1);
        }
    }
    if (tid == 0) row_parent(t, a, b, j, rp, has_u, &rs.pu, &rs.u);

    // ---- threshold: every wave's ceil(S / NW)-th largest offered code, and the
    //      least of them: at least S vectors reach it.  (Vectors past the row
    //      have code 0, below every element's.)
    const uint32_t c1 = p1.x, c2 = p1.y, c3 = p2.x, c4 = p2.y;
    const uint32_t wh = wave_kth_code<LS>(c1, c2, c3, c4, (S + NW - 1) / NW);
    const uint32_t wm = wave_max_u32(max(c1, c2));
    if (lane == 0) rs.wcode[wid] = (int)(wh | (wm << 16));
    __syncthreads();
    uint32_t h = 0xFFFFu, cmax = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t x = (uint32_t)rs.wcode[w];
        h = min(h, x & 0xFFFFu);
        cmax = max(cmax, x >> 16);
    }
    // the parent record, for the children written at the end
    const ParentRec pr = parent_rec(t, a, b, tid < K, rs.pu);

    // the row maximum (fp32: truncated); its code holds the high 16 bits alone
    const float vmax = __uint_as_float(__float_as_uint(unord32(cmax << 16)) & 0xFFFF0000u);
    // ---- candidates: elements at or above the threshold --------------------
    float tau;
    int cnt;
    // Where the threshold is no logit's (the wave with the fewest vectors has
    // not S / waves of them that are finite: supports near the number of the
    // row's vectors, masked rows) every element of the row is a candidate:
    // rows of more than fit ask the whole block's offers at once, and where
    // these bound nothing either go straight to the exact selection.
    auto unbound = [&]() { return (h << 16) <= ord32(-INFINITY) && V > CC; };
    bool again = false;
    if (unbound()) {
        h = max(h, offer_threshold<NTB>(c1, c2, c3, c4, LS, S, rs.thr));
        again = true;
    }
    for (;; again = true) {
        tau = (h << 16) > ord32(-INFINITY) ? unord32(h << 16) : -INFINITY;
        if (unbound()) {
            cnt = CC + 1;
            break;
        }
        // this thread's vectors of maximum >= tau: bit 8 bt + e is vector 2 e
        // of batch bt for e < 4, vector 2 e - 7 above (PAIR: vectors 4 e and
        // 4 e + 2 for e < 2, 4 e - 15 and 4 e - 13 for e = 4, 5).  A code >= h is a
        // maximum >= tau, except that a -0 maximum (code 0x7FFF) passes tau =
        // +0 as a logit; below the code of -inf there is only padding.
        const uint32_t hc = (h == 0x8000u) ? 0x7FFFu : max(h, 0x7Fu);
        const rs_ushort2 h2 = {(unsigned short)hc, (unsigned short)hc};
        const rs_ushort2 one = {1, 1};
        uint64_t take = 0;
        for (int bt0 = 0; bt0 < NB; bt0 += 4) {
            uint4 cw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = min(bt0 + u, NB - 1) * NTB + tid;
                if (PAIR) {
                    const uint2 x = ((const uint2*)(lds + L.codes))[i];
                    cw[u] = make_uint4(x.x, x.y, 0u, 0u);
                } else {
                    cw[u] = ((const uint4*)(lds + L.codes))[i];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t* c = &cw[u].x;
                uint32_t below = 0;
#pragma unroll
                for (int e = 0; e < (PAIR ? 2 : 4); ++e)
                    below |= __builtin_bit_cast(
                                 uint32_t, __builtin_elementwise_min(
                                               __builtin_elementwise_sub_sat(
                                                   h2, __builtin_bit_cast(rs_ushort2, c[e])),
                                               one)) << e;
                // bit e: word e's low code, bit 4 + e its high code
                const uint32_t m8 = ~((below & 0xFu) | (below >> 12)) & (PAIR ? 0x33u : 0xFFu);
                if (bt0 + u < NB) take |= (uint64_t)m8 << (8 * (bt0 + u));
            }
        }
        // in rounds of up to RND * 64 vectors per wave: listed, read, and their
        // elements >= tau appended
        int* list = (int*)s_start + wid * (WAVE * RND);
        for (;;) {
            const int tn = __popcll(take) * (PAIR ? 2 : 1);
            const int excl = wave_excl_scan(tn);
            const int total = (int)lane_u32((uint32_t)(excl + tn), WAVE - 1);
            if (total == 0) break;
            for (int pos = excl; take != 0 && pos < WAVE * RND; take &= take - 1) {
                const int bb = __builtin_ctzll(take);
                const int e = bb & 7, q0 = bb & ~7;
                if (PAIR) {
                    const int q = q0 + (e < 4 ? 4 * e : 4 * e - 15);
                    list[pos++] = rd.vidx(q);
                    list[pos++] = rd.vidx(q + 2);
                } else {
                    list[pos++] = rd.vidx(q0 + (e < 4 ? 2 * e : 2 * e - 7));
                }
            }
            wave_sync();
            uint4 x[RND];
            int e0[RND];
#pragma unroll
            for (int r = 0; r < RND; ++r) {
                x[r] = make_uint4(0, 0, 0, 0);
                e0[r] = V;
                if (r * WAVE + lane < total) {
                    const int vi = list[r * WAVE + lane];
                    x[r] = load_row_vec<DT>(rd.base, vi, V);
                    e0[r] = vi * VEC;
                }
            }
#pragma unroll
            for (int r = 0; r < RND; ++r) {
                if (r * WAVE >= total) break;
                int n = 0;
#pragma unroll
                for (int k = 0; k < VEC; ++k) n += (elem<DT>(x[r], k) >= tau) & (e0[r] + k < V);
                const int ex = wave_excl_scan(n);
                int cb = 0;
                if (lane == WAVE - 1) cb = atomicAdd(&rs.cnt, ex + n);
                int pos = (int)lane_u32((uint32_t)cb, WAVE - 1);
                if (pos > CC) take = 0;          // (too many already: the rest need not be read)
                pos += ex;
#pragma unroll
                for (int k = 0; k < VEC; ++k) {
                    const float v = elem<DT>(x[r], k);
                    if (v >= tau && e0[r] + k < V) {
                        if (pos < CC) s_keys[pos] = logit_key(v, (uint32_t)(e0[r] + k));
                        ++pos;
                    }
                }
            }
            wave_sync();
        }
        __syncthreads();
        cnt = rs.cnt;
        if (cnt <= CC || again) break;
        // Too many candidates: the row's large values are unevenly spread
        // over the lanes (sorted rows, say, or at S = 1024 one row in a hundred
        // of a Zipf prior over the ids: 2300 candidates, where S of all its
        // vectors reach a threshold of 1200).  Once more with that.
        h = codes_threshold<NTB, NBIN>((const uint32_t*)(lds + L.codes), NB * NTB * (PAIR ? 2 : 4),
                                       h, S, s_hist, rs.red, rs.thr);
        if (tid == 0) rs.cnt = 0;
        __syncthreads();
    }
    if (cnt > CC) {
        // massive ties at the threshold: exact selection from the row
        __syncthreads();
        if (tid == 0) rs.cnt = 0;
        int* const cntp = &rs.cnt;
        exact_select_fallback<DT, NTB, ROW_BATCHES * EBATCH>(
            rd.base, V, 0, h, S, CC,
            [=](float v, int id) {
                const int pos = atomicAdd(cntp, 1);
                if (pos < CC) s_keys[pos] = logit_key(v, (uint32_t)id);
            },
            &rs.cnt, rs.red, (int*)(lds + L.start));
        cnt = min(fallback_count(&rs.cnt), CC);
    }

    // ---- the support: the top S candidates in (logit desc, id asc) order ----
    // Bins linear in the value over [tau, the row maximum] (a monotone map:
    // one rounded subtraction, one rounded product).  When tau is -inf (short
    // rows, few finite logits), the upper half of the bins from the least finite
    // candidate up and the lower half linear in the id for those at -inf: by the
    // order code's high bits, an octave a bin, a level of 2000 elements, all of
    // them candidates at support 512, took 85 us, so it takes 18; with all of -inf
    // in one bin one of 1700, nine tenths masked, 100, so 20.
    const bool bounded = tau > -INFINITY;
    float low = tau, off = 0.0f;
    if (!bounded) {
        float neg = -INFINITY;                   // the largest negated value
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
            const int i = tid + r * NTB;
            const float v = key_value(s_keys[i < cnt ? i : 0]);
            if (i < cnt && v > -INFINITY) neg = fmaxf(neg, -v);
        }
        neg = wave_max(neg);
        if (lane == 0) rs.red[wid] = __float_as_int(neg);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) neg = fmaxf(neg, __int_as_float(rs.red[w]));
        low = fminf(-neg, vmax);
        off = (float)(NBIN / 2);
    }
    const float scale = fminf(((float)NBIN - off) / (vmax - low), 3e38f);
    const float per_id = (float)(NBIN / 2) / (float)V;
    uint64_t key[KPT];
    int kbin[KPT], kslot[KPT];
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int i = tid + r * NTB;
        key[r] = 0;
        kbin[r] = 0;
        kslot[r] = 0;
        if (i < cnt) {
            key[r] = s_keys[i];
            float x = (key_value(key[r]) - low) * scale + off;
            if (!bounded && !(key_value(key[r]) > -INFINITY))
                x = fminf(off - 1.0f, (float)(V - key_id(key[r])) * per_id);
            kbin[r] = (int)fminf(fmaxf(x, 0.0f), (float)(NBIN - 1));
            kslot[r] = atomicAdd(&s_hist[kbin[r]], 1);
        }
    }
    __syncthreads();
    {
        // thread tid holds bins NBIN - 1 - tid * BPT and the BPT - 1 below it;
        // a bin starts after the candidates of all higher bins
        const int top_bin = NBIN - 1 - tid * BPT;
        int hv[BPT], tot = 0;
#pragma unroll
        for (int r = 0; r < BPT; ++r) {
            hv[r] = top_bin - r >= 0 ? s_hist[top_bin - r] : 0;
            tot += hv[r];
        }
        const int ex = wave_excl_scan(tot);
        if (lane == WAVE - 1) rs.red[wid] = ex + tot;
        __syncthreads();
        int st = ex;
#pragma unroll
        for (int w = 0; w < NW; ++w) st += (w < wid) ? rs.red[w] : 0;
#pragma unroll
        for (int r = 0; r < BPT; ++r) {
            if (top_bin - r >= 0) s_start[top_bin - r] = st;
            st += hv[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        if (tid + r * NTB < cnt) {
            const int st = s_start[kbin[r]];
            if (st < S) s_ord[st + kslot[r]] = key[r];
            kslot[r] = st;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        if (tid + r * NTB < cnt && kslot[r] < S) {
            const int n = s_hist[kbin[r]];
            const uint64_t* in = s_ord + kslot[r];
            int rk = kslot[r], q = 0;
            for (; q + 4 <= n; q += 4) {
                const uint64_t k0 = in[q], k1 = in[q + 1], k2 = in[q + 2], k3 = in[q + 3];
                rk += (int)(k0 > key[r]) + (int)(k1 > key[r]) + (int)(k2 > key[r]) +
                      (int)(k3 > key[r]);
            }
            for (; q < n; ++q) rk += (int)(in[q] > key[r]);
            if (rk < S) s_top[rk] = key[r];
        }
    }
    __syncthreads();
    return RowTop{pr, vmax};
}

struct RowArgs {
    TreeDev t;
    LevelArgs a;
};

}  // namespace rheo
