// Device helpers shared by the sparse and dense pool kernels: ranking by
// counting, sums over the threads forming a pool, a child record, and the
// frontier selection of a sequence.
#pragma once

#include "rheo_device.h"
#include "rheo_state.h"

namespace rheo {

// Ranks of two keys at once (counts of larger keys among n unique keys in
// LDS, 16-byte aligned); 16 keys per step keep eight loads in flight.
__device__ __forceinline__ void count_greater2(const uint64_t* keys, int n, uint64_t k0,
                                               uint64_t k1, int& c0, int& c1) {
    const ulonglong2* kp = (const ulonglong2*)keys;
    int a0 = 0, a1 = 0;
    const int np = n >> 1;
#pragma unroll 8
    for (int j = 0; j < np; ++j) {
        const ulonglong2 x = kp[j];
        a0 += (int)(x.x > k0) + (int)(x.y > k0);
        a1 += (int)(x.x > k1) + (int)(x.y > k1);
    }
    if (n & 1) {
        const uint64_t x = keys[n - 1];
        a0 += (int)(x > k0);
        a1 += (int)(x > k1);
    }
    c0 = a0;
    c1 = a1;
}
// Ranks (counts of larger keys) of the n unique keys in LDS (16-byte
// aligned) by NT threads.  When the threads outnumber the keys, F adjacent
// lanes share a key (F a power of two, F * n <= NT, F <= 16), each counting
// over every F-th pair of keys, and their counts are added across the
// lanes; otherwise every thread ranks two keys at a time.
template <int NT>
__device__ __forceinline__ void rank_all(const uint64_t* keys, int n, int16_t* rank) {
    const int t = threadIdx.x % NT;
    int F = 1;
    while (F < 16 && 2 * F * n <= NT) F *= 2;
    if (F == 1) {
        for (int i = t; i < n; i += 2 * NT) {
            const int i2 = i + NT;
            int c0, c1;
            count_greater2(keys, n, keys[i], i2 < n ? keys[i2] : ~0ull, c0, c1);
            rank[i] = (int16_t)c0;
            if (i2 < n) rank[i2] = (int16_t)c1;
        }
        return;
    }
    const ulonglong2* kp = (const ulonglong2*)keys;
    const int i = t / F, sub = t % F;
    const uint64_t k = keys[i < n ? i : 0];
    const int np = n >> 1;
    int c = 0;
#pragma unroll 4
    for (int j = sub; j < np; j += F) {
        const ulonglong2 x = kp[j];
        c += (int)(x.x > k) + (int)(x.y > k);
    }
    if ((n & 1) && sub == 0) c += (int)(keys[n - 1] > k);
    for (int o = 1; o < F; o <<= 1) c += __shfl_xor(c, o);
    if (i < n && sub == 0) rank[i] = (int16_t)c;
}

// Sum over groups of F adjacent lanes (F = 1, 2, 4 or 8; DPP moves), in every
// lane.
__device__ __forceinline__ uint32_t lanes_sum(uint32_t x, int F) {
    if (F >= 2) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false);
    if (F >= 4) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false);
    if (F >= 8) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false);
    return x;
}

// LDS a block's pool and frontier selection exchange through.
template <int NT>
struct PoolShared {
    uint64_t w1[NT / WAVE], q[NT / WAVE];   // the waves' weight totals
    int tie[NT / WAVE];
    uint64_t s1full;                         // the row's total construction weight
    int yi;                                  // Y's place in the support
    int last;                                // the sequence's last row
    uint64_t own_score[16], own_path[16];    // the row's own children
    int own_tok[16];
};

// The parent's path score and slot path (1 and 0 for the root) and the mark
// of this level's children words, read early by the threads that later
// write the children.
struct ParentRec {
    double score;
    uint64_t path;
    uint64_t mark;
};
__device__ __forceinline__ ParentRec parent_rec(const TreeDev& t, const LevelArgs& a, int b,
                                                bool mine, int pu) {
    ParentRec p{1.0, 0ull, 0ull};
    if (a.level > 0) {
        p.mark = t.fr_mark[b];
        if (mine) {
            const Node& nd = t.node[(int64_t)b * t.NN + pu];
            p.score = nd.score;
            p.path = nd.path;
        }
    }
    return p;
}

// Children words: the fields of a level's new children that the frontier
// selection reads in another block, [B][3][NE * K]: score, slot path, token,
// each with the launch's mark in its top bit (a path is below 2^60, and a
// score's sign says nothing: it is clear, or a NaN's).  The mark flips with every launch that uses the words (the
// sequence's last row flips it once all rows have arrived), so a word that
// carries it is this launch's.  Agent-scope stores and loads.
constexpr uint64_t kMark = 1ull << 63;
__device__ __forceinline__ uint64_t* child_words(const TreeDev& t, int b) {
    return t.fr_words + (int64_t)b * 3 * t.NE * t.K;
}

// One child record of expanded row j (slot s, 0-based; App. C.1), published
// for the sequence's last row and left in LDS for this one.
// tail: the child's place in its parent's stored tail (-1: not in it)
template <int NT>
__device__ __forceinline__ void emit_child(const TreeDev& t, const LevelArgs& a, int b, int j,
                                           int pu, const ParentRec& pr, int s, int kind, int tok,
                                           double proxy, double qtrue, int tail,
                                           PoolShared<NT>& ps) {
    const int level = a.level, K = t.K;
    const int cb = (level == 0) ? 1 : 1 + K + (level - 1) * t.NE * K;
    const uint64_t score = (uint64_t)__double_as_longlong(__dmul_rn(pr.score, proxy));
    const uint64_t path = pr.path | ((uint64_t)(s + 1) << (56 - 4 * level));
    if (level > 0 && level + 1 < t.D) {
        const int n = t.NE * K;
        uint64_t* w = child_words(t, b) + j * K + s;
        __hip_atomic_store(&w[0], (score & ~kMark) | pr.mark, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&w[n], path | pr.mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&w[2 * n], (uint64_t)(uint32_t)tok | pr.mark, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    ps.own_score[s] = score;
    ps.own_path[s] = path;
    ps.own_tok[s] = tok;
    const int64_t o = (int64_t)b * t.NN + cb + j * K + s;
    Node nd;
    nd.score = __longlong_as_double((long long)score);
    nd.path = path;
    nd.meta = (level + 1) | ((s + 1) << 8) | (kind << 16);
    nd.par = pu;
    nd.tok = tok;
    nd.tidx = tail;
    nd.first_child = nd.exp_of = nd.pidx = nd.pad = -1;
    nd.proxy = proxy;
    nd.qtrue = qtrue;
    t.node[o] = nd;
    t.score[o] = nd.score;
}

// The root record (level 0 only).
__device__ __forceinline__ void emit_root(const TreeDev& t, int64_t nb) {
    Node& nd = t.node[nb];
    nd.score = 1.0;
    nd.path = 0;
    nd.meta = 0;
    nd.par = -1;
    nd.tok = -1;
    nd.tidx = -1;
    nd.proxy = 1.0;
    nd.qtrue = 1.0;
}

// The next frontier (Sec. 2.1; App. C.4, step 1).  Called by every thread of
// a row's block once wave 0 has emitted the row's children: the last row of
// sequence b to get here ranks the level's P * K new children by priority
// and keeps the best n_expand (the next level's rows take the Philox draw
// of each kept node's sampled slot themselves, keyed by this launch's
// rng_key).  s_hi and s_lo are LDS arrays of at least 256 entries the caller
// no longer needs.
//
// The arrival is not ordered after the row's children words: a word that has
// not arrived lacks the mark, and the last row reads it again (its store was
// issued before the arrival that made this row the last, so it lands whatever
// that block does next).  So nothing waits for stores to be acknowledged,
// and every row's words are read while the arrival itself is in flight.
template <int NT>
__device__ __forceinline__ void select_frontier(const TreeDev& t, const LevelArgs& a, int b,
                                                int j, const ParentRec& pr, uint64_t* s_hi,
                                                uint64_t* s_lo, PoolShared<NT>& ps) {
    __shared__ int s_tok[256];
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int level = a.level;
    const int K = t.K, NE = t.NE;
    if (level + 1 >= t.D) return;
    const int n = a.P * K;                       // <= 225 <= NT
    const int cb = (level == 0) ? 1 : 1 + K + (level - 1) * NE * K;
    const int st = NE * K;
    uint64_t* w = child_words(t, b) + tid;
    const bool other = tid < n && tid / K != j;  // a child of another row
    uint64_t x0 = 0, x1 = 0, x2 = 0;
    auto load = [&]() {
        x0 = __hip_atomic_load(&w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x1 = __hip_atomic_load(&w[st], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x2 = __hip_atomic_load(&w[2 * st], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (a.P > 1) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);  // (after the children's stores)
        uint32_t old = 0;
        if (tid == 0)
            old = __hip_atomic_fetch_add(&t.seq_cnt[b], 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        if (other) load();
        if (tid == 0) {
            ps.last = old == (uint32_t)(a.P - 1);
            if (ps.last) {
                __hip_atomic_store(&t.seq_cnt[b], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&t.fr_mark[b], pr.mark ^ kMark, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    __syncthreads();
    if (a.P > 1 && !ps.last) return;
    int tok = -1;
    uint64_t hi = 0, lo = 0;
    if (tid < n) {
        if (other) {
            for (int spin = 0; ((x0 ^ pr.mark) | (x1 ^ pr.mark) | (x2 ^ pr.mark)) & kMark; ++spin) {
                if (spin > (1 << 20)) {
                    atomicOr(t.err, 16);
                    break;
                }
                load();
            }
            tok = (int)(uint32_t)x2;
            prio_key(__longlong_as_double((long long)(x0 & ~kMark)), level + 1, x1 & ~kMark, hi, lo);
        } else {
            const int s = tid - j * K;
            tok = ps.own_tok[s];
            prio_key(__longlong_as_double((long long)ps.own_score[s]), level + 1, ps.own_path[s], hi,
                     lo);
        }
        s_hi[tid] = hi;
        s_lo[tid] = lo;
        s_tok[tid] = tok;
    } else if (tid < 256) {
        s_hi[tid] = (uint64_t)__double_as_longlong(-1.0);   // below every score
        s_lo[tid] = 0;
    }
    __syncthreads();
    // F adjacent lanes a child (a power of two, at most 8), each over every
    // F-th key.  Scores first, as the doubles they are (non-negative, not NaN:
    // prio_key; one full-rate compare).  The sampled child has its last lead's
    // score wherever that is below z, so two equal scores are the rule: the
    // places of the equal ones are summed beside their number, and of two the
    // other is known; more than two take a second pass over the keys.  Eight
    // keys are read at a time, up to the 256 that the arrays hold.
    //
    // The 144 children of twelve a node, one lane each (256 threads): read one
    // by one and in two passes they took some 7 us more than by 128-bit
    // compares in one, now less than that.
    constexpr int STEP = 8;
    int F = 1;
    while (F < 8 && 2 * F * n <= NT) F *= 2;
    const int c = tid / F;
    if (tid - lane >= n * F) return;             // whole waves past the children
    const int cc = c < n ? c : 0;
    const double mine = __longlong_as_double((long long)s_hi[cc]);
    const uint64_t mlo = s_lo[cc];
    const int ctok = s_tok[cc];
    uint32_t rk = 0, eq = 0;                     // eq: number << 16 | sum of places (< 2^16)
    for (int q = tid % F; q < n; q += STEP * F) {
        double h[STEP];
#pragma unroll
        for (int u = 0; u < STEP; ++u) h[u] = __longlong_as_double((long long)s_hi[q + u * F]);
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            rk += (uint32_t)(h[u] > mine);
            eq += h[u] == mine ? (uint32_t)(0x10000 + q + u * F) : 0u;
        }
    }
    rk = lanes_sum(rk, F);
    eq = lanes_sum(eq, F);
    if ((eq >> 16) == 2u) rk += (uint32_t)(s_lo[(int)(eq & 0xFFFFu) - cc] > mlo);
    if (__ballot((eq >> 16) > 2u) != 0ull) {
        uint32_t more = 0;
        for (int q = tid % F; q < n; q += STEP * F) {
            double h[STEP];
            uint64_t l[STEP];
#pragma unroll
            for (int u = 0; u < STEP; ++u) {
                h[u] = __longlong_as_double((long long)s_hi[q + u * F]);
                l[u] = s_lo[q + u * F];
            }
#pragma unroll
            for (int u = 0; u < STEP; ++u)
                more += (uint32_t)((int)(h[u] == mine) & (int)(l[u] > mlo));
        }
        more = lanes_sum(more, F);
        if ((eq >> 16) > 2u) rk += more;
    }
    if (tid % F == 0 && c < n && rk < (uint32_t)NE) {
        t.frontier[(int64_t)b * NE + rk] = cb + c;
        t.fr_parent[(int64_t)b * NE + rk] = c / K;
        t.fr_token[(int64_t)b * NE + rk] = ctok;
    }
}

}  // namespace rheo
