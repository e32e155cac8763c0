// Level expansion over the full vocabulary (dense mode: the support is all
// of V; Sec. 3.2 before its sparse approximation).
//
// bf16: one kernel per level, k_dense_row (described at the kernel), which
// reads each row once.  fp32, whose values hardly repeat, bf16 levels that it
// does not pay for (dense_by_rows in api.hip), and on request all: three
// kernels per level:
//  * k_select (expand.hip) with list length kk = min(V, m + K): the exact
//    top-kk of every chunk by (logit desc, id asc).
//  * k_dweights, one 256-thread block per (chunk, row): merges the row's
//    chunk lists (its top-kk by logit: the maximum M and a guess of x_{m+1}),
//    then computes for every token the construction weight w1 (relative to
//    M) and the tail weight q (relative to the guessed x_{m+1}, temperature
//    T): the chunk's sums of both, the totals of q per 64-vector sub-chunk
//    (the inverse CDF's coarse level), and a flag if a token outside the
//    top-kk ties the kk-th construction weight with a smaller id (then the
//    rank by (w1 desc, id asc) is not the rank by logit).
//  * k_dpool, one 256-thread block per row: ranks the top-kk by (w1 desc, id
//    asc) -- exactly, by a row scan, when flagged -- checks the guess of
//    x_{m+1} (recomputing the tail totals when it was wrong), removes the
//    leads from the tail, samples Y by inverse CDF over token ids (sub-chunk
//    totals, then one re-read sub-chunk), forms the pool (App. C.1) and
//    stores what verification needs (Z_q, the logit of x_{m+1}, the leads).
//    Then the frontier selection shared with the sparse pool.
#include "rheo_device.h"
#include "rheo_state.h"
#include "pool_common.h"
#include "row_select.h"

namespace rheo {

constexpr int NTD = 256;
constexpr int KKMAX = 32;         // m + K <= 29
constexpr int DLIST_MAX = 512;    // C * kk keys a row's chunk lists hold
constexpr int NCHMAX = 1024;      // sub-chunks per row: V <= 262143, >= 256 tokens each

// Vector vi of a row, elements past V as -inf: of weight 0, without a test.
template <int DT>
__device__ __forceinline__ uint4 dload_vec(const char* base, int vi, int V) {
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
            const uint32_t lo = (e0 < V) ? p16[e0] : 0xFF80u;
            const uint32_t hi = (e0 + 1 < V) ? p16[e0 + 1] : 0xFF80u;
            w[q] = lo | (hi << 16);
        }
    } else {
        const uint32_t* p32 = (const uint32_t*)base;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (e + q < V) ? p32[e + q] : 0xFF800000u;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

template <int DT>
__device__ __forceinline__ float dlogit(const char* row, int v) {
    if (DT) return __uint_as_float((uint32_t)((const uint16_t*)row)[v] << 16);
    return ((const float*)row)[v];
}

// The row's top-kk by logit key from its C chunk lists (unique keys; 0 marks
// an empty slot), into s_tl[0..kk).  All threads of the block take part.
__device__ __forceinline__ void row_top_by_logit(const TreeDev& t, int row, uint64_t* s_list,
                                                 uint64_t* s_tl) {
    const int kk = t.Sc, nl = t.C * kk;
    const uint64_t* src = t.sel + (int64_t)row * nl;
    for (int i = threadIdx.x; i < nl; i += blockDim.x) s_list[i] = src[i];
    __syncthreads();
    for (int i = threadIdx.x; i < nl; i += blockDim.x) {
        const uint64_t k = s_list[i];
        if (k == 0ull) continue;
        int rk = 0;
        for (int q = 0; q < nl; ++q) rk += (int)(s_list[q] > k);
        if (rk < kk) s_tl[rk] = k;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// k_dweights: weights, sums and sub-chunk totals of one chunk of one row
// ---------------------------------------------------------------------------
template <int DT, int NVC>
__global__ __launch_bounds__(NTD) void k_dweights(TreeDev t, LevelArgs a) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int ESZ = DT ? 2 : 4;
    __shared__ uint64_t s_list[DLIST_MAX];
    __shared__ uint64_t s_tl[KKMAX];
    __shared__ uint32_t s_tw[KKMAX];
    __shared__ uint64_t s_red[NTD / WAVE];
    __shared__ float s_M, s_ref;
    __shared__ uint32_t s_wmin;
    __shared__ uint64_t s_kb;
    __shared__ int s_idmax;

    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int c = blockIdx.x, row = blockIdx.y;
    const int V = t.V, m = t.m, kk = t.Sc;
    const int v0 = c * NTD * NVC;
    const char* base = (const char*)a.logits + (int64_t)row * t.stride * ESZ;

    uint4 r[NVC];
#pragma unroll
    for (int i = 0; i < NVC; ++i) r[i] = dload_vec<DT>(base, v0 + i * NTD + tid, V);

    row_top_by_logit(t, row, s_list, s_tl);
    if (tid < kk) s_tw[tid] = cweight(key_value(s_tl[tid]), key_value(s_tl[0]), a.k1);
    __syncthreads();
    if (tid == 0) {
        s_M = key_value(s_tl[0]);
        s_ref = key_value(s_tl[m]);                    // guess of x_{m+1}
        const uint32_t wmin = s_tw[kk - 1];
        int idmax = -1;
        for (int i = 0; i < kk; ++i)
            if (s_tw[i] == wmin) idmax = max(idmax, key_id(s_tl[i]));
        s_wmin = wmin;
        s_kb = s_tl[kk - 1];
        s_idmax = idmax;
    }
    __syncthreads();
    const float M = s_M, ref = s_ref;
    const uint32_t wmin = s_wmin;
    const uint64_t kb = s_kb;
    const int idmax = s_idmax;

    // Per element: w1 relative to the row maximum (never above it, so no
    // upper clamp), q relative to the guess of x_{m+1}; weights are summed
    // in pairs in 32 bits (each <= 2^30) before the 64-bit totals.  Each
    // vector's q total goes to LDS, and the totals of the sub-chunks (64
    // consecutive vectors: one wave's at one step) are formed there.  A
    // weight equal to the kk-th one is only marked per element; the exact
    // test of the rank tie runs for the marked elements alone (rare).
    uint64_t s1 = 0, zq = 0;
    bool flag = false;
    constexpr int NG = NVC < 16 ? NVC : 16;          // vectors per LDS round
    __shared__ uint64_t s_vq[NG][NTD];
    for (int g0 = 0; g0 < NVC; g0 += NG) {
#pragma unroll
        for (int ii = 0; ii < NG; ++ii) {
            const int i = g0 + ii;
            const int e0 = (v0 + i * NTD + tid) * VEC;
            // (elements past V read as -inf: weight 0 on both counts, and
            // no tie, since idmax < V)
            uint64_t sq = 0;
            uint32_t hit = 0;
#pragma unroll
            for (int k = 0; k < VEC; k += 2) {
                const float la = elem<DT>(r[i], k), lb = elem<DT>(r[i], k + 1);
                const uint32_t wa = cweight_below(la, M, a.k1);
                const uint32_t wb = cweight_below(lb, M, a.k1);
                s1 += (uint64_t)(wa + wb);
                sq += (uint64_t)(cweight(la, ref, a.kT) + cweight(lb, ref, a.kT));
                hit |= (uint32_t)(wa == wmin) << k;
                hit |= (uint32_t)(wb == wmin) << (k + 1);
            }
            if (hit) {
#pragma unroll
                for (int k = 0; k < VEC; ++k) {
                    const int id = e0 + k;
                    if (((hit >> k) & 1u) && id < idmax &&
                        logit_key(elem<DT>(r[i], k), (uint32_t)id) < kb)
                        flag = true;
                }
            }
            zq += sq;
            s_vq[ii][tid] = sq;
        }
        __syncthreads();
        // sub-chunk (ii, wave w): lanes 64 w .. 64 w + 63 of row ii, summed
        // by 4 threads of 16 entries each
        for (int q = tid; q < NG * (NTD / WAVE) * 4; q += NTD) {
            const int part = q & 3, sc = q >> 2;
            const int ii = sc / (NTD / WAVE), w = sc % (NTD / WAVE);
            uint64_t x = 0;
#pragma unroll
            for (int l = 0; l < 16; ++l) x += s_vq[ii][w * WAVE + part * 16 + l];
            x += __shfl_xor(x, 1);
            x += __shfl_xor(x, 2);
            const int sub = (v0 + (g0 + ii) * NTD) / WAVE + w;
            if (part == 0 && sub < t.NCH) t.dq[(int64_t)row * t.NCH + sub] = x;
        }
        __syncthreads();
    }
    s1 = block_sum_u64<NTD>(s1, s_red);
    zq = block_sum_u64<NTD>(zq, s_red);
    if (__syncthreads_or(flag) && tid == 0) atomicOr(&t.dflag[row], 1);
    if (tid == 0) {
        t.dpart[((int64_t)row * t.C + c) * 2 + 0] = s1;
        t.dpart[((int64_t)row * t.C + c) * 2 + 1] = zq;
    }
}

// A token outside the top kk by logit ties the kk-th construction weight with a
// smaller id.  The top kk by (w1, id) is then: every token with w1 above that
// weight (all among the top kk by logit), and the lowest ids with exactly that
// weight, found by a scan of the row in id order, a vector a thread at a time and
// no further than the last of them.  s_tl: the top kk by logit; s_rk: their keys
// w1 << 32 | ~id.
template <int DT, int NT>
__device__ __noinline__ void ranks_by_weight(const char* base, int V, float M, float k1, int kk,
                                             const uint64_t* s_tl, const uint64_t* s_rk,
                                             uint64_t* s_x, uint32_t* s_xw, uint64_t* s_red) {
    constexpr int VEC = DT ? 8 : 4;
    const int tid = threadIdx.x;
    uint32_t wmin = 0xFFFFFFFFu;
    for (int q = 0; q < kk; ++q) wmin = min(wmin, (uint32_t)(s_rk[q] >> 32));
    int ngt = 0;
    for (int q = 0; q < kk; ++q) ngt += (int)((uint32_t)(s_rk[q] >> 32) > wmin);
    const int need = kk - ngt;
    // the tokens above wmin keep their (w1, id) order first
    if (tid < kk && (uint32_t)(s_rk[tid] >> 32) > wmin) {
        const uint64_t k = s_rk[tid];
        int rk = 0;
        for (int q = 0; q < kk; ++q) rk += (int)(s_rk[q] > k);
        s_x[rk] = s_tl[tid];
        s_xw[rk] = (uint32_t)(k >> 32);
    }
    int before = 0;                              // tokens of weight wmin so far
    for (int v0 = 0; v0 * VEC < V && before < need; v0 += NT) {
        const uint4 x = dload_vec<DT>(base, v0 + tid, V);
        const int e0 = (v0 + tid) * VEC;
        uint32_t hit = 0;
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            hit |= (uint32_t)(e0 + k < V && cweight(elem<DT>(x, k), M, k1) == wmin) << k;
        uint64_t tot;
        int pos = before + (int)block_excl_scan_u64<NT>((uint64_t)__popc(hit), s_red, &tot);
        if (hit != 0u && pos < need) {
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                if (((hit >> k) & 1u) == 0u) continue;
                if (pos < need) {
                    s_x[ngt + pos] = logit_key(elem<DT>(x, k), (uint32_t)(e0 + k));
                    s_xw[ngt + pos] = wmin;
                }
                ++pos;
            }
        }
        before += (int)tot;
    }
}

// ---------------------------------------------------------------------------
// k_dpool: ranks, tail, Y, pool and frontier of one row
// ---------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(NTD) void k_dpool(TreeDev t, LevelArgs a) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int ESZ = DT ? 2 : 4;
    constexpr int CHT = WAVE * VEC;              // tokens per sub-chunk
    __shared__ uint64_t s_list[DLIST_MAX];
    __shared__ uint64_t s_tl[KKMAX];             // top-kk by logit key
    __shared__ uint64_t s_x[KKMAX];              // x_1..x_kk (logit keys) by (w1 desc, id asc)
    __shared__ uint32_t s_xw[KKMAX];             // their construction weights
    __shared__ uint64_t s_rk[KKMAX];             // ranking keys (w1 << 32 | ~id)
    __shared__ uint64_t s_sub[NCHMAX];           // tail totals per sub-chunk
    __shared__ uint64_t s_cq[CHT];               // tail weights of one sub-chunk
    __shared__ uint64_t s_red[NTD / WAVE];
    __shared__ PoolShared<NTD> ps;
    __shared__ int s_pu, s_cs, s_y, s_flag;
    __shared__ uint64_t s_u, s_t2, s_qy;

    const int tid = threadIdx.x, lane = tid % WAVE;
    const int row = blockIdx.x;
    const int b = row / a.P, j = row % a.P;
    const int V = t.V, K = t.K, m = t.m, kk = t.Sc, C = t.C, NE = t.NE, NCH = t.NCH;
    const int level = a.level;
    const int64_t nb = (int64_t)b * t.NN;
    const char* base = (const char*)a.logits + (int64_t)row * t.stride * ESZ;

    if (tid == 0) {
        int pu = (level == 0) ? 0 : t.frontier[(int64_t)b * NE + j];
        const int lo_uid = (level == 0) ? 0 : ((level == 1) ? 1 : 1 + K + (level - 2) * NE * K);
        const int hi_uid = (level == 0) ? 1 : lo_uid + ((level == 1) ? 1 : NE) * K;
        bool bad = pu < lo_uid || pu >= hi_uid;
        if (bad) {
            atomicOr(t.err, 16);
            pu = 0;
        }
        s_pu = pu;
        // the draw of the parent's sampled slot, keyed by the launch that
        // created the parent
        s_u = philox_draw((level == 0 || bad) ? a.rng_key : a.fr_key, P_DRAFT, (uint64_t)b,
                          (uint64_t)pu);
        s_flag = t.dflag[row];
        t.dflag[row] = 0;                        // clean for the next level
        s_y = -1;
        s_cs = -1;
    }
    // the row's construction and tail totals and its sub-chunk tail totals
    // (relative to the guess of x_{m+1}), loaded now: they arrive while the
    // top of the row is ranked
    uint64_t S1 = 0, Zq = 0;
    for (int c = 0; c < C; ++c) {
        S1 += t.dpart[((int64_t)row * C + c) * 2 + 0];
        Zq += t.dpart[((int64_t)row * C + c) * 2 + 1];
    }
    uint64_t dqv[NCHMAX / NTD];
#pragma unroll
    for (int q = 0; q < NCHMAX / NTD; ++q) {
        const int i = tid + q * NTD;
        dqv[q] = (i < NCH) ? t.dq[(int64_t)row * NCH + i] : 0ull;
    }
    row_top_by_logit(t, row, s_list, s_tl);
    const ParentRec pr = parent_rec(t, a, b, tid < K, s_pu);
    const float M = key_value(s_tl[0]);

    // x_1..x_kk by (w1 desc, id asc)
    if (!s_flag) {
        if (tid < kk) {
            const uint32_t w = cweight(key_value(s_tl[tid]), M, a.k1);
            s_rk[tid] = ((uint64_t)w << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)key_id(s_tl[tid]));
        }
        __syncthreads();
        if (tid < kk) {
            const uint64_t k = s_rk[tid];
            int rk = 0;
            for (int q = 0; q < kk; ++q) rk += (int)(s_rk[q] > k);
            s_x[rk] = s_tl[tid];
            s_xw[rk] = (uint32_t)(k >> 32);
        }
    } else {
        if (tid < kk) {
            const uint32_t w = cweight(key_value(s_tl[tid]), M, a.k1);
            s_rk[tid] = ((uint64_t)w << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)key_id(s_tl[tid]));
        }
        __syncthreads();
        ranks_by_weight<DT, NTD>(base, V, M, a.k1, kk, s_tl, s_rk, s_x, s_xw, s_red);
    }
    __syncthreads();

    // x_{m+1} and the tail totals
    const float ref_t = key_value(s_x[m]);
    if (tid == 0 && !(ref_t > -INFINITY)) atomicOr(t.err, 512);   // x_{m+1} is -inf
    const int nch = NCH;
    if (ref_t == key_value(s_tl[m])) {
#pragma unroll
        for (int q = 0; q < NCHMAX / NTD; ++q)
            if (tid + q * NTD < nch) s_sub[tid + q * NTD] = dqv[q];
    } else {
        // the guess of x_{m+1} was wrong (construction-weight ties): tail
        // totals again, relative to the right logit, one sub-chunk per wave
        // pass
        uint64_t part = 0;
        for (int i = tid / WAVE; i < nch; i += NTD / WAVE) {
            const int v0 = i * CHT + lane * VEC;
            uint64_t sq = 0;
            for (int k = 0; k < VEC; ++k)
                if (v0 + k < V) sq += cweight(dlogit<DT>(base, v0 + k), ref_t, a.kT);
            const uint64_t ws = wave_sum_u64(sq);
            if (lane == 0) s_sub[i] = ws;
            part += (lane == 0) ? ws : 0ull;
        }
        Zq = block_sum_u64<NTD>(part, s_red);
    }
    __syncthreads();
    // the leads leave the tail
    uint64_t lead_q = 0;
    for (int i = 0; i < m; ++i) lead_q += cweight(key_value(s_x[i]), ref_t, a.kT);
    if (tid == 0) {
        for (int i = 0; i < m; ++i) {
            const int id = key_id(s_x[i]);
            s_sub[id / CHT] -= cweight(key_value(s_x[i]), ref_t, a.kT);
        }
    }
    Zq -= lead_q;
    __syncthreads();

    // Y ~ q~_T: t = floor(U64 Zq / 2^64), the sub-chunk holding t, then the
    // first token of it whose inclusive prefix exceeds the remainder
    {
        const uint64_t tt = __umul64hi(s_u, Zq);
        const int cpt = (nch + NTD - 1) / NTD;
        const int ca = min(nch, tid * cpt), cz = min(nch, ca + cpt);
        uint64_t mysum = 0;
        for (int i = ca; i < cz; ++i) mysum += s_sub[i];
        uint64_t tot;
        uint64_t acc = block_excl_scan_u64<NTD>(mysum, s_red, &tot);
        if (acc <= tt && tt < acc + mysum) {
            for (int i = ca; i < cz; ++i) {
                if (tt < acc + s_sub[i]) {
                    s_cs = i;
                    s_t2 = tt - acc;
                    break;
                }
                acc += s_sub[i];
            }
        }
        __syncthreads();
        const int cs = s_cs;
        if (cs < 0) {
            if (tid == 0) atomicOr(t.err, 1);
        } else {
            for (int i = tid; i < CHT; i += NTD) {
                const int v = cs * CHT + i;
                uint64_t w = 0;
                if (v < V) {
                    w = cweight(dlogit<DT>(base, v), ref_t, a.kT);
                    for (int q = 0; q < m; ++q)
                        if (key_id(s_x[q]) == v) w = 0;
                }
                s_cq[i] = w;
            }
            __syncthreads();
            constexpr int TPT = CHT / NTD;       // tokens per thread (1 or 2)
            uint64_t mine = 0;
#pragma unroll
            for (int q = 0; q < TPT; ++q) mine += s_cq[tid * TPT + q];
            uint64_t acc2 = block_excl_scan_u64<NTD>(mine, s_red, &tot);
            const uint64_t t2 = s_t2;
            if (acc2 <= t2 && t2 < acc2 + mine) {
#pragma unroll
                for (int q = 0; q < TPT; ++q) {
                    const uint64_t w = s_cq[tid * TPT + q];
                    if (t2 < acc2 + w) {
                        s_y = cs * CHT + tid * TPT + q;
                        s_qy = w;
                        break;
                    }
                    acc2 += w;
                }
            }
        }
        __syncthreads();
    }
    int ytok = s_y;
    uint64_t qy = s_qy;
    if (ytok < 0) {                              // unreachable fallback
        if (tid == 0) atomicOr(t.err, 1);
        ytok = key_id(s_x[m]);
        qy = 1;
    }

    // the K children: top-m leads, Y, fills (App. C.1)
    const int pu = s_pu;
    const int cb = (level == 0) ? 1 : 1 + K + (level - 1) * NE * K;
    const int e_idx = (level == 0) ? 0 : 1 + (level - 1) * NE + j;
    if (tid == 0) {
        t.zq[(int64_t)b * t.E + e_idx] = Zq;
        t.dref[(int64_t)b * t.E + e_idx] = ref_t;
        for (int i = 0; i < m; ++i) t.dleads[((int64_t)b * t.E + e_idx) * 16 + i] = key_id(s_x[i]);
        t.node[nb + pu].first_child = cb + j * K;
        t.node[nb + pu].exp_of = e_idx;
        if (level == 0) emit_root(t, nb);
    }
    if (tid < K) {
        const int s = tid;
        int yr = kk;                             // Y's place among x_{m+1}.. (kk: beyond)
        for (int q = m; q < kk; ++q)
            if (key_id(s_x[q]) == ytok) yr = q;
        int kind, tok;
        double proxy;
        const double dS1 = (double)S1;
        if (s < m || t.topk) {                   // a lead (pure top-K pools: every slot)
            kind = LEAD;
            tok = key_id(s_x[s]);
            proxy = __ddiv_rn((double)s_xw[s], dS1);
        } else if (s == m) {
            kind = SAMPLED;
            tok = ytok;
            if (m >= 1) {
                uint64_t lead = 0;
                for (int q2 = 0; q2 < m; ++q2) lead += s_xw[q2];
                const uint64_t z = S1 - lead;
                const uint64_t wm = s_xw[m - 1];
                proxy = __ddiv_rn((double)(wm < z ? wm : z), dS1);
            } else {
                proxy = fmin(1.0, __dadd_rn(__ddiv_rn((double)s_xw[0], dS1), t.eps));
            }
        } else {
            const int f = s - m - 1;
            const int rk = m + f + ((m + f) >= yr ? 1 : 0);
            kind = FILL;
            tok = key_id(s_x[rk]);
            proxy = __ddiv_rn((double)s_xw[rk], dS1);
        }
        const double qtrue = (kind == SAMPLED) ? __ddiv_rn((double)qy, (double)Zq) : proxy;
        emit_child(t, a, b, j, pu, pr, s, kind, tok, proxy, qtrue, -1, ps);
    }
    // the next frontier: the last row of the sequence to finish selects it
    select_frontier(t, a, b, j, pr, s_sub, s_sub + 256, ps);
}

// ---------------------------------------------------------------------------
// k_dense_row: the whole level for one bf16 row per 512-thread block, the row
// read once.
//
// While the row streams its values are counted (code_hist.h), one table per
// batch of 32768 elements, and its top m + K found (row_top).  The weights of
// the counted values, each evaluated once, times the counts give the total
// construction weight and every batch's tail weight; the tail weight of each
// value then replaces the counts in the first two tables.  Y ~ q~_T lies in
// the batch whose interval holds t = floor(U64 Zq / 2^64), which alone is read
// again: its weights come from the tables.
//
// Where the counts do not cover the row (a value of 2^9 or more, a weight
// below -2^9, an overflow, more small values than are listed, few values) the
// sums and Y's batch take every element's own weight, in one more pass over the
// row.  Where a value outside the top m + K shares the last one's construction
// weight, the ranks come from a scan of the row in id order.
//
// Evaluating both weights of every element in a pass of its own bound the
// level (30 vector instructions an element): at 512 rows of 128256, 34 us to
// select, 60 for the weights and 15 for the pools, against 56 here.
// ---------------------------------------------------------------------------
constexpr int NTX = 512;

__global__ __launch_bounds__(NTX, 4) void k_dense_row(RowArgs) {
    constexpr int NW = NTX / WAVE;
    constexpr int SEGV = NTX * EBATCH;           // vectors of a batch
    const RowArgs& args = kernel_params<RowArgs>();
    const TreeDev& t = args.t;
    const LevelArgs& a = args.a;
    extern __shared__ __align__(16) uint8_t s_pdyn[];
    __shared__ RowShared<NTX> rs;
    __shared__ PoolShared<NTX> ps;
    __shared__ uint64_t s_x[KKMAX];              // x_1..x_kk (logit keys) by (w1 desc, id asc)
    __shared__ uint32_t s_xw[KKMAX];             // their construction weights
    __shared__ uint64_t s_rk[KKMAX];             // ranking keys (w1 << 32 | ~id)
    __shared__ uint64_t s_seg[ROW_BATCHES];      // the batches' tail weights
    __shared__ uint64_t s_w1, s_n, s_qy;
    __shared__ uint64_t s_slot[NW];              // the waves' tail weights of a batch
    __shared__ uint64_t s_red[NW];
    __shared__ int s_flag, s_y, s_idmax;

    ieee_mode_off();                             // NaN words drop out of the maxima
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int row = blockIdx.x;
    const int b = row / a.P, j = row % a.P;
    const int V = t.V, K = t.K, m = t.m, kk = t.Sc, NE = t.NE;
    const int level = a.level;
    const int64_t nb = (int64_t)b * t.NN;
    const int NB = row_batches<1, NTX>(V);
    const RowLds L = row_lds(kk, false, NB, NTX, COUNT_BATCH);
    uint64_t* s_top = (uint64_t*)(s_pdyn + L.p.top);
    uint32_t* tab = (uint32_t*)(s_pdyn + L.tab);
    const uint32_t* s_small = (const uint32_t*)(s_pdyn + L.small);
    const RowReader<1, NTX> rd = row_reader<1, NTX>(t, a, row);
    if (tid < ROW_BATCHES) s_seg[tid] = 0;
    if (tid == 0) {
        s_w1 = 0;
        s_n = 0;
        s_flag = 0;
        s_y = -1;
        s_idmax = -1;
    }
    const RowTop rt = row_top<1, false, NTX, COUNT_BATCH>(t, a, row, kk, s_pdyn, L, rd, rs);

    // ---- the sums, relative to M and to the guess x_{m+1} = s_top[m] --------
    const float M = key_value(s_top[0]);
    const float guess = key_value(s_top[m]);
    const uint64_t kb = s_top[kk - 1];
    const float vb = key_value(kb);
    const uint32_t wmin = cweight(vb, M, a.k1);  // the least weight of the top kk
    const int ns = rs.nsmall;
    // (NS: the tables read, 4 or 8)
    auto totals = [&](auto NS_) {
        constexpr int NS = decltype(NS_)::value;
        uint64_t w1 = 0, n = 0, zq[NS];
        bool tie = false;
#pragma unroll
        for (int s = 0; s < NS; ++s) zq[s] = 0;
        for (int i = tid; i < HIST_WORDS; i += NTX) {
            uint32_t c[NS], any = 0, pos = 0, neg = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                c[s] = s < NB ? tab[s * HIST_WORDS + i] : 0u;
                any |= c[s];
                pos += c[s] & 0xFFFFu;
                neg += c[s] >> 16;
            }
            n += pos + neg;
            uint32_t qp = 0, qn = 0;
            if (i >= 1 && i < HIST_OUT) {
                if (pos) {
                    const float l = hist_value(i);
                    const uint32_t w = cweight(l, M, a.k1);
                    qp = cweight(l, guess, a.kT);
                    tie |= l < vb && w == wmin;
                    w1 += (uint64_t)pos * w;
#pragma unroll
                    for (int s = 0; s < NS; ++s) zq[s] += (uint64_t)(c[s] & 0xFFFFu) * qp;
                }
                if (neg) {
                    const float l = -hist_value(i);
                    const uint32_t w = cweight(l, M, a.k1);
                    qn = cweight(l, guess, a.kT);
                    tie |= l < vb && w == wmin;
                    w1 += (uint64_t)neg * w;
#pragma unroll
                    for (int s = 0; s < NS; ++s) zq[s] += (uint64_t)(c[s] >> 16) * qn;
                }
            } else if (i == 0) {
                // zeros, and the listed values, which are put right below
                const uint32_t w = cweight(0.0f, M, a.k1);
                qp = qn = cweight(0.0f, guess, a.kT);
                tie |= pos + neg > (uint32_t)ns && 0.0f < vb && w == wmin;
                w1 += (uint64_t)(pos + neg) * w;
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    zq[s] += (uint64_t)((c[s] & 0xFFFFu) + (c[s] >> 16)) * qp;
            } else {
                // -2^9 and below: only if of no weight
                if (pos || (neg && (cweight(-512.0f, M, a.k1) != 0u ||
                                    cweight(-512.0f, guess, a.kT) != 0u)))
                    n += 1ull << 40;
                tie |= any != 0 && wmin == 0u;
            }
            // the tail weight of each value, where its counts were
            tab[i] = qp;
            tab[HIST_WORDS + i] = qn;
        }
        for (int i = tid; i < ns; i += NTX) {
            const float l = __uint_as_float(s_small[i] << 16);
            const uint32_t w = cweight(l, M, a.k1);
            w1 += (uint64_t)w - cweight(0.0f, M, a.k1);
            tie |= l < vb && w == wmin;
            atomicAdd((unsigned long long*)&s_seg[s_small[i] >> 16],
                      (unsigned long long)((uint64_t)cweight(l, guess, a.kT) -
                                           cweight(0.0f, guess, a.kT)));
        }
        // two different logits of the list that share its last weight
        if (tid < kk) {
            const uint64_t k = s_top[tid];
            tie |= (k >> 32) != (kb >> 32) && cweight(key_value(k), M, a.k1) == wmin;
        }
        w1 = wave_sum_u64(w1);
        n = wave_sum_u64(n);
        if (lane == 0) {
            atomicAdd((unsigned long long*)&s_w1, (unsigned long long)w1);
            atomicAdd((unsigned long long*)&s_n, (unsigned long long)n);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint64_t z = wave_sum_u64(zq[s]);
            if (lane == 0 && s < NB)
                atomicAdd((unsigned long long*)&s_seg[s], (unsigned long long)z);
        }
        if (__ballot(tie) != 0ull && lane == 0) s_flag = 1;
    };
    if (ns <= HIST_SMALL) {
        if (NB <= 4) totals(std::integral_constant<int, 4>());
        else totals(std::integral_constant<int, ROW_BATCHES>());
    }
    // x_1..x_kk by (w1 desc, id asc): ranks among the top kk by logit
    if (tid < kk) {
        const uint32_t w = cweight(key_value(s_top[tid]), M, a.k1);
        s_rk[tid] = ((uint64_t)w << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)key_id(s_top[tid]));
        if (w == wmin) atomicMax(&s_idmax, key_id(s_top[tid]));
    }
    __syncthreads();
    bool counted = ns <= HIST_SMALL && s_n == (uint64_t)(NB * NTX) * (EBATCH * 8);
    uint64_t S1 = s_w1;
    float ref_t = guess;
    for (bool direct = !counted;;) {
        if (direct) {
            // every element's own weights, relative to M and to ref_t, and whether one
            // past the top kk ties the last construction weight with a smaller id
            const int idmax = s_idmax;
            bool tie = false;
            S1 = 0;
            for (int s = 0; s < NB; ++s) {
                uint64_t w1 = 0, zq = 0;
                uint4 next = dload_vec<1>(rd.base, rd.vidx(s * EBATCH), V);
#pragma unroll 1
                for (int q = s * EBATCH; q < (s + 1) * EBATCH; ++q) {
                    const uint4 x = next;
                    const int e0 = rd.vidx(q) * 8;
                    if (q + 1 < (s + 1) * EBATCH)
                        next = dload_vec<1>(rd.base, rd.vidx(q + 1), V);
                    if (e0 >= V) continue;
                    uint32_t hit = 0;
#pragma unroll
                    for (int k = 0; k < 8; k += 2) {
                        // (elements past V read as -inf: weight 0 on both counts)
                        const float la = elem<1>(x, k), lb = elem<1>(x, k + 1);
                        const uint32_t wa = cweight_below(la, M, a.k1);
                        const uint32_t wb = cweight_below(lb, M, a.k1);
                        w1 += (uint64_t)(wa + wb);
                        zq += (uint64_t)(cweight(la, ref_t, a.kT) + cweight(lb, ref_t, a.kT));
                        hit |= (uint32_t)(wa == wmin) << k;
                        hit |= (uint32_t)(wb == wmin) << (k + 1);
                    }
                    if (hit) {
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            tie |= ((hit >> k) & 1u) && e0 + k < idmax &&
                                   logit_key(elem<1>(x, k), (uint32_t)(e0 + k)) < kb;
                    }
                }
                S1 += block_sum_u64<NTX>(w1, s_red);
                zq = block_sum_u64<NTX>(zq, s_red);
                if (tid == 0) s_seg[s] = zq;
            }
            if (tid == 0) s_flag = 0;            // (what incomplete counts may have set)
            __syncthreads();
            if (__ballot(tie) != 0ull && lane == 0) s_flag = 1;
            __syncthreads();
            if (ref_t != guess) break;           // (the ranks are known)
        }
        if (!s_flag) {
            if (tid < kk) {
                const uint64_t k = s_rk[tid];
                int rk = 0;
                for (int q = 0; q < kk; ++q) rk += (int)(s_rk[q] > k);
                s_x[rk] = s_top[tid];
                s_xw[rk] = (uint32_t)(k >> 32);
            }
        } else {
            ranks_by_weight<1, NTX>(rd.base, V, M, a.k1, kk, s_top, s_rk, s_x, s_xw, s_red);
        }
        __syncthreads();
        const float ref = key_value(s_x[m]);
        if (ref == guess) break;
        // the guess of x_{m+1} was wrong (construction-weight ties): the sums again
        ref_t = ref;
        counted = false;
        direct = true;
    }
    if (tid == 0 && !(ref_t > -INFINITY)) atomicOr(t.err, 512);   // x_{m+1} is -inf

    // ---- Y ~ q~_T: the leads leave the tail; the batch that holds
    //      t = floor(U64 Zq / 2^64), then the 64-vector slot, then the token
    uint64_t Zq = 0;
    for (int s = 0; s < NB; ++s) Zq += s_seg[s];
    for (int i = 0; i < m; ++i) Zq -= cweight(key_value(s_x[i]), ref_t, a.kT);
    int cs = -1;
    uint64_t t2 = 0;
    {
        const uint64_t tt = __umul64hi(rs.u, Zq);
        uint64_t acc = 0;
        for (int s = 0; s < NB; ++s) {
            uint64_t z = s_seg[s];
            for (int i = 0; i < m; ++i)
                if (key_id(s_x[i]) / (SEGV * 8) == s) z -= cweight(key_value(s_x[i]), ref_t, a.kT);
            if (cs < 0 && tt < acc + z) {
                cs = s;
                t2 = tt - acc;
            }
            acc += z;
        }
    }
    if (cs >= 0) {
        // wave w reads the 64-vector slots 8 w .. 8 w + 7 of the batch
        const int v0 = cs * SEGV + wid * (EBATCH * WAVE) + lane;
        uint4 r[EBATCH];
#pragma unroll
        for (int e = 0; e < EBATCH; ++e) r[e] = load_row_vec<1>(rd.base, v0 + e * WAVE, V);
        uint64_t sq[EBATCH], all = 0;
        const hist_u16x2 hbase = {(unsigned short)HIST_BASE, (unsigned short)HIST_BASE};
        const hist_u16x2 hout = {(unsigned short)HIST_OUT, (unsigned short)HIST_OUT};
        const hist_u16x2 four = {4, 4};
        const hist_u16x2 half = {(unsigned short)HIST_BYTES, (unsigned short)HIST_BYTES};
#pragma unroll
        for (int e = 0; e < EBATCH; ++e) {
            const uint32_t* w = &r[e].x;
            sq[e] = 0;
            if (counted) {
                // the value's weight from the tables (word 0: that of zeros, which
                // other values below 2^-11 put right; past the row NaN words, of
                // no weight)
                hist_u16x2 least = {0xFFFF, 0xFFFF};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const hist_u16x2 mag = __builtin_bit_cast(hist_u16x2, w[c] & 0x7FFF7FFFu);
                    hist_u16x2 i = __builtin_elementwise_sub_sat(mag, hbase);
                    least = __builtin_elementwise_min(least, i);
                    i = __builtin_elementwise_min(i, hout) * four +
                        (__builtin_bit_cast(hist_u16x2, w[c]) >> (unsigned short)15) * half;
                    sq[e] += (uint64_t)(*(const uint32_t*)((const uint8_t*)tab + i.x) +
                                        *(const uint32_t*)((const uint8_t*)tab + i.y));
                }
                if (__ballot(least.x == 0 || least.y == 0) != 0ull &&
                    __ballot(hist_has_small(hist_least_less_1(r[e]))) != 0ull) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        for (int k = 0; k < 2; ++k) {
                            const uint32_t bits = (w[c] >> (16 * k)) & 0xFFFFu;
                            if ((bits & 0x7FFFu) - 1u < HIST_BASE)
                                sq[e] += (uint64_t)cweight(__uint_as_float(bits << 16), ref_t, a.kT) -
                                         tab[0];
                        }
                }
            } else {
                const int e0 = (v0 + e * WAVE) * 8;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    sq[e] += (e0 + k < V) ? cweight(elem<1>(r[e], k), ref_t, a.kT) : 0u;
            }
            for (int i = 0; i < m; ++i)
                if (key_id(s_x[i]) / 8 == v0 + e * WAVE)
                    sq[e] -= cweight(key_value(s_x[i]), ref_t, a.kT);
            all += sq[e];
            __builtin_amdgcn_sched_barrier(0);   // (one vector's lookups in registers at a time)
        }
        all = wave_sum_u64(all);
        if (lane == 0) s_slot[wid] = all;
        __syncthreads();
        // the wave that holds t2 goes through its slots, then the lanes of one
        uint64_t acc = 0;
        int own = -1;
        for (int w = 0; w < NW; ++w) {
            const uint64_t z = s_slot[w];
            if (own < 0 && t2 - acc < z) own = w;
            if (own < 0) acc += z;
        }
        if (own == wid) {
            uint64_t t3 = t2 - acc;              // remainder within the slots to come
            uint64_t p = 0, mine = 0;
            int slot = -1;
#pragma unroll
            for (int e = 0; e < EBATCH; ++e) {
                if (slot < 0) {
                    const uint64_t inc = wave_incl_scan_u64(sq[e]);
                    const uint64_t z = lane_u64(inc, WAVE - 1);
                    if (t3 >= z) {
                        t3 -= z;
                    } else {
                        slot = e;
                        p = inc - sq[e];
                        mine = sq[e];
                    }
                }
            }
            if (slot >= 0 && p <= t3 && t3 - p < mine) {
                // one lane: its vector again, element by element
                const int vi = v0 + slot * WAVE;
                const uint4 x = load_row_vec<1>(rd.base, vi, V);
                bool found = false;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    uint64_t q = vi * 8 + k < V ? cweight(elem<1>(x, k), ref_t, a.kT) : 0u;
                    for (int i = 0; i < m; ++i)
                        if (key_id(s_x[i]) == vi * 8 + k) q = 0;
                    if (!found && t3 < p + q) {
                        found = true;
                        s_y = vi * 8 + k;
                        s_qy = q;
                    }
                    p += q;
                }
            }
        }
    }
    __syncthreads();

    // ---- wave 0: the expanded node's record and its K children (App. C.1) ----
    if (wid == 0) {
        int ytok = s_y;
        uint32_t qy = (uint32_t)s_qy;
        if (ytok < 0) {                          // unreachable fallback
            if (tid == 0) atomicOr(t.err, 1);
            ytok = key_id(s_x[m]);
            qy = 1;
        }
        const int pu = rs.pu;
        const int cb = (level == 0) ? 1 : 1 + K + (level - 1) * NE * K;
        const int e_idx = (level == 0) ? 0 : 1 + (level - 1) * NE + j;
        if (tid == 0) {
            t.zq[(int64_t)b * t.E + e_idx] = Zq;
            t.dref[(int64_t)b * t.E + e_idx] = ref_t;
            t.node[nb + pu].first_child = cb + j * K;
            t.node[nb + pu].exp_of = e_idx;
            if (level == 0) emit_root(t, nb);
        }
        if (tid < m) t.dleads[((int64_t)b * t.E + e_idx) * 16 + tid] = key_id(s_x[tid]);
        // Y's place among x_{m+1}.. (kk: beyond)
        const uint64_t at = __ballot(tid >= m && tid < kk && key_id(s_x[min(tid, kk - 1)]) == ytok);
        const int yr = at ? (int)__builtin_ctzll(at) : kk;
        int rk = min(tid, kk - 1), kind = LEAD;  // pure top-K pools: every slot a lead
        if (!t.topk && tid >= m) {
            kind = tid == m ? SAMPLED : FILL;
            rk = min(tid - 1 + (tid - 1 >= yr ? 1 : 0), kk - 1);
        }
        if (kind == SAMPLED) rk = 0;
        // one division for all lanes, Y's own probability in lane 32
        uint32_t num = s_xw[max(rk, 0)];
        uint64_t den = S1;
        if (kind == SAMPLED && m >= 1) {
            uint64_t lead = 0;
            for (int q = 0; q < m; ++q) lead += s_xw[q];
            const uint64_t z = S1 - lead;
            const uint64_t wm = s_xw[m - 1];
            num = (uint32_t)(wm < z ? wm : z);
        }
        if (lane == 32) {
            num = qy;
            den = Zq;
        }
        double proxy = __ddiv_rn((double)num, (double)den);
        const uint64_t py = lane_u64((uint64_t)__double_as_longlong(proxy), 32);
        if (kind == SAMPLED && m == 0) proxy = fmin(1.0, __dadd_rn(proxy, t.eps));
        const double qtrue = kind == SAMPLED ? __longlong_as_double((long long)py) : proxy;
        const int tok = kind == SAMPLED ? ytok : key_id(s_x[max(rk, 0)]);
        if (tid < K) emit_child(t, a, b, j, pu, rt.pr, tid, kind, tok, proxy, qtrue, -1, ps);
    }
    select_frontier(t, a, b, j, rt.pr, s_top, (uint64_t*)(s_pdyn + L.p.k2), ps);
}

static size_t dense_row_shm(const TreeDev& t) {
    return (size_t)row_lds(t.Sc, false, row_batches<1, NTX>(t.V), NTX, COUNT_BATCH).p.bytes;
}

// Raises the kernel's limit on dynamic LDS.
hipError_t prepare_dense(const TreeDev& t) {
    if (!t.dense || !t.dtype) return hipSuccess;
    if (dense_row_shm(t) > kRowLdsMax) return hipErrorInvalidValue;
    return hipFuncSetAttribute((const void*)&k_dense_row,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRowLdsMax);
}

hipError_t launch_dense_row(const TreeDev& t, const LevelArgs& a, hipStream_t s) {
    RowArgs ra{t, a};
    ra.a.cached = level_cached(t, t.B * a.P);
    void* args[] = {&ra};
    return hipLaunchKernel((const void*)&k_dense_row, dim3(t.B * a.P), dim3(NTX), args,
                           dense_row_shm(t), s);
}

template <int DT>
static void launch_dense_dt(const TreeDev& t, const LevelArgs& a, int nvc, int rows,
                            hipStream_t s) {
    const dim3 grid(t.C, rows);
    switch (nvc) {
    case 4: k_dweights<DT, 4><<<grid, NTD, 0, s>>>(t, a); break;
    case 8: k_dweights<DT, 8><<<grid, NTD, 0, s>>>(t, a); break;
    case 16: k_dweights<DT, 16><<<grid, NTD, 0, s>>>(t, a); break;
    default: k_dweights<DT, 32><<<grid, NTD, 0, s>>>(t, a); break;
    }
    k_dpool<DT><<<rows, NTD, 0, s>>>(t, a);
}

hipError_t launch_dense(const TreeDev& t, const LevelArgs& a, int nvc, hipStream_t s) {
    const int rows = t.B * a.P;
    if (t.dtype) launch_dense_dt<1>(t, a, nvc, rows, s);
    else launch_dense_dt<0>(t, a, nvc, rows, s);
    return hipGetLastError();
}

}  // namespace rheo
