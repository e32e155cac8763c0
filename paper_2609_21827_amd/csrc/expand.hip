// Level expansion of the draft tree: top-S selection over each draft-logit
// row, the node's distributions, the hybrid candidate pool with its proxy
// and true probabilities, and the parent each row belongs to.
//
// One kernel per level, k_expand_row: one block per row (described at the
// kernel).  Where a row's LDS does not fit it (fp32 rows of some 230,000 elements
// and more with supports above some 290), or on request, two kernels:
//  * k_select, one 256-thread block per (chunk, row): the chunk is streamed
//    from HBM into registers with 16-byte loads and its exact top-Sc by
//    (logit desc, id asc) is written, sorted, to the tree's selection
//    scratch (Sc = S: a chunk is larger than any support).  The row's top-S
//    lies in the union of its chunks' top-S.  Within a chunk, a value that
//    Sc per-vector maxima reach is a threshold at least Sc elements reach,
//    so the chunk's top-Sc are among the few elements at or above it; they
//    are collected in LDS and ranked exactly.  (Dense mode's lists come from
//    it too.)
//  * k_pool, one 256-thread block per row: takes the row's parent from the
//    stored frontier and merges the chunk lists into the row's top-S support
//    (Sec. 3.2, sparse draft distributions).
// Both end with the pool (Sec. 3.2; App. C.1): construction weights q
// (untempered, Sec. 5.4), ranks by (q desc, id asc), the tail q~_T = q_T / z
// on the support minus the top-m, Y ~ q~_T by inverse CDF over the ranked
// tail, fills, proxies (min{q(x_m), z}; q(x_1) + eps for m = 0), the true
// probability q~(Y), path scores (App. C.1).  The last row of a sequence to
// finish (an arrival counter) ranks the level's new children by priority
// and stores the n_expand best, which the next level's rows expand (Sec.
// 2.1; App. C.4, step 1).  Children fields pass between blocks only through
// agent-coherent atomic stores and loads (pool_common.h).
#include "rheo_device.h"
#include "rheo_state.h"
#include "pool_common.h"
#include "row_select.h"

namespace rheo {

constexpr int NTC = 256;      // threads per k_select block
constexpr int NTP = 256;      // threads per k_pool block
constexpr int CAPC = 1024;    // candidates a chunk collects in LDS
constexpr int CAPV = 512;     // candidate vectors a chunk collects in LDS
constexpr int MERGE_MAX = 2048;  // chunk-list keys one row merges (C * Sc)
// ---------------------------------------------------------------------------
// the pool of one row: parent, support, distributions and children
// ---------------------------------------------------------------------------
// The pool of one row from its support s_top (App. C.1), formed by NT
// threads, EPT consecutive support entries each (S <= NT * EPT).  A support
// slot left empty (no candidate reached it) is flagged and taken as -inf.
//
// It is a chain of dependent steps (latency, not throughput, bounds it), so
// it has two exchanges in all: one for both weight totals, the masses
// before every entry and the weight ties, one for Y; the sums run as 32-bit
// scans of the weights' 16-bit halves (a DPP add per step); the children's
// probabilities and Y's come from one division (Y's in a lane of its own).
// At V = 128256, S = 128 (clock stamps): 7200 cycles before these, 5400 now.
template <int NT, int EPT>
__device__ __forceinline__ void pool_form(const TreeDev& t, const LevelArgs& a, int row,
                                          uint8_t* lds, const PoolLds& L, int pu,
                                          const ParentRec& pr, uint64_t u, PoolShared<NT>& ps) {
    constexpr int NW = NT / WAVE;
    uint64_t* s_top = (uint64_t*)(lds + L.top);
    uint64_t* s_k2 = (uint64_t*)(lds + L.k2);
    uint32_t* s_w1 = (uint32_t*)(lds + L.w1);
    uint32_t* s_q = (uint32_t*)(lds + L.q);
    int16_t* s_wr = (int16_t*)(lds + L.wr);
    int16_t* s_xs = (int16_t*)(lds + L.xs);
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int b = row / a.P;
    const int j = row % a.P;
    const int S = t.S, K = t.K, m = t.m;
    const int level = a.level;
    const int NE = t.NE;
    const int64_t nb = (int64_t)b * t.NN;
    const int cb = (level == 0) ? 1 : 1 + K + (level - 1) * NE * K;
    const int e_idx = (level == 0) ? 0 : 1 + (level - 1) * NE + j;
    if (tid == 0) ps.yi = -1;

    // Construction weights w1 (untempered unless asked) and, taking the rank
    // by (w1 desc, id asc) to be the support order, the tail weights of q~_T
    // relative to x_{m+1} = s_top[m].  The support is in (logit desc, id asc)
    // order and the weight never grows along it, so the rank differs from the
    // position only where two different logits share a weight: then the ranks
    // and the tail are computed again.
    //
    // The tail, x_{m+1} .. x_S in rank order, is written to the tree in that
    // order (token, q~ weight) for verification, and Y ~ q~_T is the entry
    // whose interval [mass before, mass before + q) holds
    // t = floor(U64 Zq / 2^64): the inverse CDF over the tail in rank order.
    auto filled = [&](uint64_t k) {
        return (uint32_t)key_id(k) >= (uint32_t)t.V ? logit_key(-INFINITY, 0u) : k;
    };
    const float M = key_value(filled(s_top[0]));
    const float ref0 = key_value(filled(s_top[m]));
    const int i0 = tid * EPT;
    uint64_t ek[EPT];
    uint32_t eq[EPT];
    uint64_t pre;                                // tail mass of the wave before this thread's
    bool tie = false;
    {
        uint32_t w1lo = 0, w1hi = 0, qlo = 0, qhi = 0;
        uint64_t kp = filled(s_top[i0 > 0 && i0 < S ? i0 - 1 : 0]);
        uint32_t wp = cweight(key_value(kp), M, a.k1);
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
            const int i = i0 + r;
            ek[r] = 0;
            eq[r] = 0;
            if (i < S) {
                const uint64_t raw = s_top[i];
                ek[r] = filled(raw);
                if (raw != ek[r]) atomicOr(t.err, 256);     // a support slot left empty
                const float v = key_value(ek[r]);
                const uint32_t w = cweight(v, M, a.k1);
                const uint32_t q = (i >= m) ? cweight(v, ref0, a.kT) : 0u;
                tie |= i > 0 && w == wp && (ek[r] >> 32) != (kp >> 32);
                kp = ek[r];
                wp = w;
                s_w1[i] = w;
                s_q[i] = q;
                eq[r] = q;
                w1lo += w & 0xFFFFu;
                w1hi += w >> 16;
                qlo += q & 0xFFFFu;
                qhi += q >> 16;
            }
        }
        // inclusive scans over the wave (sums of at most 256 halves: < 2^24)
        w1lo = wave_incl_scan_u32(w1lo);
        w1hi = wave_incl_scan_u32(w1hi);
        const uint32_t mlo = qlo, mhi = qhi;
        qlo = wave_incl_scan_u32(qlo);
        qhi = wave_incl_scan_u32(qhi);
        const uint64_t anytie = __ballot(tie);
        if (lane == WAVE - 1) {
            ps.w1[wid] = ((uint64_t)w1hi << 16) + w1lo;
            ps.q[wid] = ((uint64_t)qhi << 16) + qlo;
            ps.tie[wid] = anytie != 0ull;
        }
        pre = ((uint64_t)(qhi - mhi) << 16) + (qlo - mlo);
    }
    __syncthreads();
    uint64_t S1 = 0, Zq = 0;
    int anyt = 0;
    const int nwa = (S + WAVE * EPT - 1) / (WAVE * EPT);    // waves that hold entries
    for (int w = 0; w < nwa; ++w) {
        S1 += ps.w1[w];
        const uint64_t zw = ps.q[w];
        Zq += zw;
        pre += (w < wid) ? zw : 0ull;
        anyt |= ps.tie[w];
    }
    if (t.cfull) S1 = ps.s1full;             // construction over the whole vocabulary
    const int64_t tail_base = ((int64_t)b * t.E + e_idx) * S;
    const bool ident = anyt == 0;
    if (ident) {
        const uint64_t tt = __umul64hi(u, Zq);
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
            const int i = i0 + r;
            if (i >= m && i < S) {
                t.tail_id[tail_base + i - m] = key_id(ek[r]);
                t.tail_q[tail_base + i - m] = eq[r];
                if (pre <= tt && tt - pre < (uint64_t)eq[r]) ps.yi = i;
                pre += eq[r];
            }
        }
    } else {
        // two different logits share a weight: ranks by (w1 desc, id asc), the
        // tail relative to the right x_{m+1}, contiguous runs of ranks per
        // thread and a block scan of their masses
        __syncthreads();
        for (int i = tid; i < S; i += NT)
            s_k2[i] = ((uint64_t)s_w1[i] << 32) |
                      (uint64_t)(0xFFFFFFFFu - (uint32_t)key_id(filled(s_top[i])));
        __syncthreads();
        rank_all<NT>(s_k2, S, s_wr);
        __syncthreads();
        for (int i = tid; i < S; i += NT) s_xs[s_wr[i]] = (int16_t)i;
        __syncthreads();
        const float ref_t = key_value(filled(s_top[s_xs[m]]));
        uint64_t partq = 0;
        for (int i = tid; i < S; i += NT) {
            const uint32_t q = (s_wr[i] >= m) ? cweight(key_value(filled(s_top[i])), ref_t, a.kT) : 0u;
            s_q[i] = q;
            partq += q;
        }
        Zq = block_sum_u64<NT>(partq, ps.q);
        const uint64_t tt = __umul64hi(u, Zq);
        const int ntail = S - m;
        const int per = (ntail + NT - 1) / NT;
        const int r0 = min(S, m + tid * per), r1 = min(S, r0 + per);
        uint64_t mine = 0;
        for (int r = r0; r < r1; ++r) mine += s_q[s_xs[r]];
        uint64_t tot;
        uint64_t acc = block_excl_scan_u64<NT>(mine, ps.q, &tot);
        for (int r = r0; r < r1; ++r) {
            const int i = s_xs[r];
            const uint32_t q = s_q[i];
            t.tail_id[tail_base + r - m] = key_id(filled(s_top[i]));
            t.tail_q[tail_base + r - m] = q;
            if (acc <= tt && tt - acc < (uint64_t)q) ps.yi = i;
            acc += q;
        }
    }
    __syncthreads();
    if (wid != 0) return;

    // ---- wave 0: the expanded node's record and its K children -------------
    // position in the support of rank r, and rank of position i
    auto xs = [&](int r) -> int { return ident ? r : (int)s_xs[r]; };
    auto wr = [&](int i) -> int { return ident ? i : (int)s_wr[i]; };
    int yi = ps.yi;
    if (yi < 0) {
        if (tid == 0) atomicOr(t.err, 1);
        yi = xs(m);                              // unreachable fallback
    }
    if (tid == 0) {
        // q~_T is taken relative to x_{m+1}: undefined when its logit is
        // -inf (fewer than m + 1 tokens of the support above the rest)
        if (!(key_value(filled(s_top[xs(m)])) > -INFINITY)) atomicOr(t.err, 512);
        t.zq[(int64_t)b * t.E + e_idx] = Zq;
        t.node[nb + pu].first_child = cb + j * K;
        t.node[nb + pu].exp_of = e_idx;
        if (level == 0) emit_root(t, nb);
    }
    // top-m leads, Y, fills (App. C.1); pure top-K pools: the K best by (w1
    // desc, id asc)
    int item = yi, kind = SAMPLED;
    if (t.topk || tid < m) {
        item = xs(min(tid, S - 1));
        kind = LEAD;
    } else if (tid != m && tid < K) {
        const int rk = tid - 1;                  // Y itself is passed over
        item = xs(rk + (rk >= wr(yi) ? 1 : 0));
        kind = FILL;
    }
    // one division for all lanes: lane s < K its child's proxy w1 / S1 (the
    // sampled child: min{w1(x_m), z} / S1, for m = 0 w1(x_1) / S1 + eps),
    // lane 32 the sampled child's probability q / Zq
    uint32_t num = s_w1[item];
    uint64_t den = S1;
    if (kind == SAMPLED) {
        num = s_w1[xs(0)];
        if (m >= 1) {
            uint64_t lead = 0;
            for (int q2 = 0; q2 < m; ++q2) lead += s_w1[xs(q2)];
            const uint64_t z = S1 - lead;
            const uint64_t wm = s_w1[xs(m - 1)];
            num = (uint32_t)(wm < z ? wm : z);
        }
    }
    if (lane == 32) {
        num = s_q[yi];
        den = Zq;
    }
    double proxy = __ddiv_rn((double)num, (double)den);
    const uint64_t py = lane_u64((uint64_t)__double_as_longlong(proxy), 32);
    if (kind == SAMPLED && m == 0) proxy = fmin(1.0, __dadd_rn(proxy, t.eps));
    const double qtrue = (kind == SAMPLED) ? __longlong_as_double((long long)py) : proxy;
    if (tid < K)
        emit_child(t, a, b, j, pu, pr, tid, kind, key_id(filled(s_top[item])), proxy, qtrue,
                   wr(item) >= m ? wr(item) - m : -1, ps);
}

// ---------------------------------------------------------------------------
// k_pool: one block per row: parent, support (merge of the chunk lists),
// pool, and, by the last row of each sequence, the next frontier
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NTP) void k_pool(TreeDev t, LevelArgs a) {
    extern __shared__ __align__(16) uint8_t s_pdyn[];
    __shared__ PoolShared<NTP> ps;
    __shared__ int s_pu;
    __shared__ uint64_t s_u;
    const PoolLds L = pool_lds(t.S, t.C);
    uint64_t* s_m = (uint64_t*)(s_pdyn + L.m);    // the C chunk lists, C * S keys
    uint64_t* s_top = (uint64_t*)(s_pdyn + L.top);
    uint64_t* s_k2 = (uint64_t*)(s_pdyn + L.k2);

    const int tid = threadIdx.x;
    const int row = blockIdx.x;
    const int b = row / a.P;
    const int j = row % a.P;
    const int S = t.S, K = t.K;
    const int C = t.C;
    const int level = a.level;
    const int NE = t.NE;
    const int64_t nb = (int64_t)b * t.NN;

    // the parent: frontier node j of the previous level (the n_expand
    // children with the highest priority, chosen by the previous launch)
    // with the Philox draw of its sampled slot; and the chunk lists, with
    // an empty list after them
    const int C4 = (C + 3) & ~3;
    if (tid == 0) row_parent(t, a, b, j, row_parent_load(t, a, b, j), false, &s_pu, &s_u);
    const uint64_t* src = t.sel + (int64_t)row * C * S;
    for (int i = tid; i < C * S; i += NTP) s_m[i] = src[i];
    for (int i = C * S + tid; i < (C + 1) * S; i += NTP) s_m[i] = 0ull;
    for (int i = tid; i < S; i += NTP) s_top[i] = 0ull;   // id -1 until merged
    __syncthreads();
    // the parent record, for the children written at the end
    const ParentRec pr = parent_rec(t, a, b, tid < K, s_pu);

    // merge: a key's rank in the row is its position in its own (sorted)
    // list plus the count of larger keys in every other list (a binary
    // search per list).  Every list holds S keys (a chunk is larger than any
    // support); keys are unique and 0 marks an empty slot.  Two keys per
    // thread and four lists at a time (the empty list stands in for lists
    // past the last), with no branches, keep eight loads in flight per
    // search step.
    {
        int pw2 = 1;
        while (pw2 * 2 <= S) pw2 *= 2;
        const int nk = C * S;
        for (int eA = tid; eA < nk; eA += 2 * NTP) {
            const int eB = eA + NTP;
            const uint64_t kA = s_m[eA], kB = eB < nk ? s_m[eB] : 0ull;
            const int lA = eA / S, lB = eB / S;
            int rA = eA - lA * S, rB = eB - lB * S;
            for (int c2 = 0; c2 < C4; c2 += 4) {
                int lb[4];
#pragma unroll
                for (int cc = 0; cc < 4; ++cc) lb[cc] = min(c2 + cc, C) * S;
                int oA[4] = {0, 0, 0, 0}, oB[4] = {0, 0, 0, 0};
                for (int half = pw2; half > 0; half >>= 1) {
                    uint64_t xA[4], xB[4];
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) {
                        xA[cc] = s_m[lb[cc] + min(oA[cc] + half, S) - 1];
                        xB[cc] = s_m[lb[cc] + min(oB[cc] + half, S) - 1];
                    }
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) {
                        oA[cc] += (oA[cc] + half <= S && xA[cc] > kA) ? half : 0;
                        oB[cc] += (oB[cc] + half <= S && xB[cc] > kB) ? half : 0;
                    }
                }
#pragma unroll
                for (int cc = 0; cc < 4; ++cc) {
                    rA += (c2 + cc != lA) ? oA[cc] : 0;
                    rB += (c2 + cc != lB) ? oB[cc] : 0;
                }
            }
            if (kA != 0ull && rA < S) s_top[rA] = kA;
            if (kB != 0ull && rB < S) s_top[rB] = kB;
        }
    }
    __syncthreads();

    // the pool, formed by the whole block
    if (t.cfull && tid == 0) ps.s1full = t.s1row[row];   // (read past pool_form's first barrier)
    if (S <= NTP) pool_form<NTP, 1>(t, a, row, s_pdyn, L, s_pu, pr, s_u, ps);
    else pool_form<NTP, SMAX / NTP>(t, a, row, s_pdyn, L, s_pu, pr, s_u, ps);

    // the next frontier: the last row of the sequence to finish selects it
    select_frontier(t, a, b, j, pr, s_top, s_k2, ps);
}

// ---------------------------------------------------------------------------
// k_select: the exact top-Sc of one chunk of one row
// ---------------------------------------------------------------------------
// A bf16 chunk holds at most 65536 elements, so its candidates are ranked by
// 32-bit keys: the 16-bit order code of the value above the complement of
// the chunk-local index (larger key = larger logit, then smaller id).  fp32
// chunks use the 64-bit row keys.
__device__ __forceinline__ uint32_t chunk_key32(float v, int lid) {
    return (ord32(v) & 0xFFFF0000u) | (uint32_t)(0xFFFF - lid);
}
// The row key (logit_key) of a chunk key; e0 = the chunk's first element.
__device__ __forceinline__ uint64_t row_key_of32(uint32_t k, int e0) {
    const uint32_t o = (k & 0xFFFF0000u) | ((k & 0x80000000u) ? 0u : 0xFFFFu);
    const uint32_t id = (uint32_t)(e0 + 0xFFFF - (int)(k & 0xFFFFu));
    return ((uint64_t)o << 32) | (uint64_t)(0xFFFFFFFFu - id);
}

template <int NT>
__device__ void rank_keys32(const uint32_t* keys, int n, int16_t* rank) {
    int npad = 1;
    while (npad < n) npad <<= 1;
    int F = NT / npad;
    if (F < 1) F = 1;
    if (F > WAVE) F = WAVE;
    const int sub = threadIdx.x % F;
    const int per = NT / F;
    const uint4* k4 = (const uint4*)keys;
    const int n4 = n >> 2;
    for (int base = 0; base < n; base += per) {
        const int i = base + threadIdx.x / F;
        int cnt = 0;
        if (i < n) {
            const uint32_t k = keys[i];
#pragma unroll 4
            for (int g = sub; g < n4; g += F) {
                const uint4 x = k4[g];
                cnt += (int)(x.x > k) + (int)(x.y > k) + (int)(x.z > k) + (int)(x.w > k);
            }
            for (int j = 4 * n4 + sub; j < n; j += F) cnt += (int)(keys[j] > k);
        }
        for (int o = 1; o < F; o <<= 1) cnt += __shfl_xor(cnt, o);
        if (i < n && sub == 0) rank[i] = (int16_t)cnt;
    }
}

template <int DT, int NVC>
__device__ __forceinline__ void select_block(const TreeDev& t, const LevelArgs& a) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int NM = DT ? (NVC + 1) / 2 : NVC;   // registers of per-vector maxima
    constexpr int NW = NTC / WAVE;
    constexpr int WCAP = CAPV / NW;                // candidate vectors per wave

    __shared__ __align__(16) uint64_t s_keys[CAPC];   // candidates (bf16: 32-bit keys)
    __shared__ uint4 s_cv[CAPV];                 // candidate vectors, WCAP per wave
    __shared__ int16_t s_rank[CAPC];
    __shared__ int s_cvi[CAPV];                  // their vector indices
    __shared__ int s_thr[2 * NW * 16];          // threshold counts
    __shared__ int s_bc[2][NW];
    __shared__ int s_wn[NW];
    __shared__ int s_cnt;
    __shared__ int s_redi[NW];
    uint32_t* s_k32 = (uint32_t*)s_keys;

    ieee_mode_off();                             // NaN words drop out of the maxima
    const int tid = threadIdx.x;
    const int lane = tid % WAVE, wid = tid / WAVE;
    const int c = blockIdx.x;
    const int row = blockIdx.y;
    const int V = t.V;
    const int v0 = c * NTC * NVC;                           // first vector of the chunk
    const int nvalid = min(V - v0 * VEC, NTC * NVC * VEC);  // >= 1: C = ceil(V / chunk)
    const int nsel = min(t.Sc, nvalid);
    const int NVR = (V + VEC - 1) / VEC;                    // vectors of the row
    const char* base = (const char*)a.logits + (int64_t)row * t.stride * (DT ? 2 : 4);
    uint64_t* out = t.sel + ((int64_t)row * t.C + c) * t.Sc;

    // the chunk, NVC 16-byte vectors per thread; every chunk but a row's
    // last is whole, so its loads need no bounds checks
    uint4 r[NVC];
    if ((v0 + NTC * NVC) * VEC <= V) {
        const uint32_t toff = (uint32_t)tid * 16u;
#pragma unroll
        for (int i = 0; i < NVC; ++i)
            r[i] = load_stream16(base + (int64_t)(v0 + i * NTC) * 16 + toff);
    } else {
#pragma unroll
        for (int i = 0; i < NVC; ++i) r[i] = load_row_vec<DT>(base, v0 + i * NTC + tid, V);
    }
    if (tid == 0) s_cnt = 0;

    // per-vector maxima (exact; bf16: two per register, high halves) and
    // every thread's two largest as 16-bit order codes
    uint32_t vm[NM];
    uint32_t c1 = 0, c2 = 0;
    if (DT) {
        rs_ushort2 p1 = {0, 0}, p2 = {0, 0};
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const uint32_t lo = bf16x8_max_raw(r[2 * q]);
            const uint32_t hi = (2 * q + 1 < NVC) ? bf16x8_max_raw(r[2 * q + 1]) : lo;
            vm[q] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
            const rs_ushort2 cq = bf16x2_codes(vm[q]);
            p2 = __builtin_elementwise_max(p2, __builtin_elementwise_min(p1, cq));
            p1 = __builtin_elementwise_max(p1, cq);
        }
        c1 = max((uint32_t)p1.x, (uint32_t)p1.y);
        c2 = max(min((uint32_t)p1.x, (uint32_t)p1.y), max((uint32_t)p2.x, (uint32_t)p2.y));
    } else {
#pragma unroll
        for (int i = 0; i < NVC; ++i) {
            const float mx = fmaxf(fmaxf(elem<DT>(r[i], 0), elem<DT>(r[i], 1)),
                                   fmaxf(elem<DT>(r[i], 2), elem<DT>(r[i], 3)));
            vm[i] = __float_as_uint(mx);
            const uint32_t cv = ord32(mx) >> 16;
            c2 = max(c2, min(c1, cv));
            c1 = max(c1, cv);
        }
    }

    // threshold tau: at least nsel elements of the chunk are >= tau.  Every
    // thread offers the order codes of its two largest vector maxima; h =
    // the nsel-th largest offered code gives tau = the smallest value with
    // code h (each offered maximum is a distinct vector holding an element
    // >= tau), found four bits at a time (offer_threshold).  Elements past
    // the row end read as -inf (fp32) or a NaN word (bf16), so in a row's
    // last chunk tau may fall to -inf; vectors wholly past the row end are
    // never candidates, so the candidates are then the chunk's valid
    // elements.  Supports larger than the offers use all vector maxima.
    static_assert(NTC == 256, "one histogram bin per thread");
    uint32_t h = 0;
    if (nsel <= 2 * NTC) {
        h = offer_threshold<NTC>(c1, c2, nsel, s_thr);
    } else {
#pragma unroll 1
        for (int bit = 15; bit >= 0; --bit) {
            const uint32_t cand = h | (1u << bit);
            int n = 0;
#pragma unroll
            for (int i = 0; i < NVC; ++i) {
                const float v = DT ? ((i & 1) ? bf_hi(vm[i / 2]) : bf_lo(vm[i / 2]))
                                   : __uint_as_float(vm[i]);
                n += (ord32(v) >> 16) >= cand;
            }
            n = wave_sum_i32(n);
            if (lane == 0) s_bc[bit & 1][wid] = n;
            __syncthreads();
            int tot = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) tot += s_bc[bit & 1][w];
            if (tot >= nsel) h = cand;
        }
    }
    const float tau = (h << 16) > ord32(-INFINITY) ? unord32(h << 16) : -INFINITY;

    // candidates >= tau in two compactions, so the per-element work touches
    // only the few vectors whose maximum reaches tau: (1) every wave appends
    // its candidate vectors to its own LDS region (ballot and bit count);
    // (2) the threads take the candidate vectors of all regions in turn and
    // append their elements >= tau to the candidate list.  If a wave has more
    // candidate vectors than its region holds, but all fit, they are written
    // again into one list with slots reserved per wave; more than that sends
    // the chunk to the exact fallback below.
    {
        int wpos = 0;
#pragma unroll
        for (int i = 0; i < NVC; ++i) {
            const float vmax = DT ? ((i & 1) ? bf_hi(vm[i / 2]) : bf_lo(vm[i / 2]))
                                  : __uint_as_float(vm[i]);
            const bool take = vmax >= tau && v0 + i * NTC + tid < NVR;
            const uint64_t msk = __ballot(take);
            if (take) {
                const int pos = wpos + (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(msk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)msk, 0u));
                if (pos < WCAP) {
                    s_cv[wid * WCAP + pos] = r[i];
                    s_cvi[wid * WCAP + pos] = v0 + i * NTC + tid;
                }
            }
            wpos += __popcll(msk);
        }
        if (lane == 0) s_wn[wid] = wpos;
    }
    __syncthreads();
    int wn[NW], nv = 0, wbefore = 0;
    bool ovf = false;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wn[w] = s_wn[w];
        ovf |= wn[w] > WCAP;
        wbefore += (w < wid) ? wn[w] : 0;
        nv += wn[w];
    }
    const bool contig = ovf && nv <= CAPV;
    if (contig) {
        // one list: each wave's vectors after those of the waves before it
        int wpos = wbefore;
#pragma unroll
        for (int i = 0; i < NVC; ++i) {
            const float vmax = DT ? ((i & 1) ? bf_hi(vm[i / 2]) : bf_lo(vm[i / 2]))
                                  : __uint_as_float(vm[i]);
            const bool take = vmax >= tau && v0 + i * NTC + tid < NVR;
            const uint64_t msk = __ballot(take);
            if (take) {
                const int pos = wpos + (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(msk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)msk, 0u));
                s_cv[pos] = r[i];
                s_cvi[pos] = v0 + i * NTC + tid;
            }
            wpos += __popcll(msk);
        }
        __syncthreads();
    }
    if (!ovf || contig) {
        for (int j0 = 0; j0 < nv; j0 += NTC) {
            const int j = j0 + tid;
            // entry j of the concatenated regions (or of the one list)
            int w = 0, off = j;
            if (!contig) {
#pragma unroll
                for (int q = 0; q < NW - 1; ++q) {
                    const bool past = off >= wn[q] && w == q;
                    off -= past ? wn[q] : 0;
                    w += past ? 1 : 0;
                }
            }
            uint4 x = make_uint4(0, 0, 0, 0);
            int e0 = V;
            if (j < nv) {
                x = s_cv[w * WCAP + off];
                e0 = s_cvi[w * WCAP + off] * VEC;
            }
            int n = 0;
#pragma unroll
            for (int k = 0; k < VEC; ++k) n += (elem<DT>(x, k) >= tau) & (e0 + k < V);
            const int excl = wave_excl_scan(n);
            int cbase = 0;
            if (lane == WAVE - 1) cbase = atomicAdd(&s_cnt, excl + n);
            int pos = (int)lane_u32((uint32_t)cbase, WAVE - 1) + excl;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                const float v = elem<DT>(x, k);
                if (v >= tau && e0 + k < V) {
                    if (pos < CAPC) {
                        if (DT) s_k32[pos] = chunk_key32(v, e0 + k - v0 * VEC);
                        else s_keys[pos] = logit_key(v, (uint32_t)(e0 + k));
                    }
                    ++pos;
                }
            }
        }
    } else if (tid == 0) {
        s_cnt = CAPC + 1;                        // too many: exact fallback below
    }
    __syncthreads();
    int cnt = s_cnt;

    if (cnt > CAPC) {
        // degenerate chunk: exact selection from the chunk in memory
        const int eb = v0 * VEC;                 // first element of the chunk
        __shared__ int s_scr[256];           // (32 vectors x NW waves, or a digit's counts)
        __syncthreads();
        if (tid == 0) s_cnt = 0;
        exact_select_fallback<DT, NTC, NVC>(
            base, V, v0, h, nsel, CAPC,
            [&](float v, int id) {
                const int pos = atomicAdd(&s_cnt, 1);
                if (pos < CAPC) {
                    if (DT) s_k32[pos] = chunk_key32(v, id - eb);
                    else s_keys[pos] = logit_key(v, (uint32_t)id);
                }
            },
            &s_cnt, s_redi, s_scr);
        cnt = min(fallback_count(&s_cnt), CAPC);
    }

    // exact top-nsel of the candidates, written sorted; unused slots are 0
    // (below every real key)
    if (DT) rank_keys32<NTC>(s_k32, cnt, s_rank);
    else rank_keys<NTC>(s_keys, cnt, s_rank);
    __syncthreads();
    for (int i = tid; i < cnt; i += NTC) {
        const int rk = s_rank[i];
        if (rk < nsel) out[rk] = DT ? row_key_of32(s_k32[i], v0 * VEC) : s_keys[i];
    }
    for (int i = nsel + tid; i < t.Sc; i += NTC) out[i] = 0ull;
}


// ---------------------------------------------------------------------------
// k_expand_row: the whole level for one row per block: the row's support
// (row_top), the pool (App. C.1) and, by the last row of each sequence, the
// next frontier.
//
// LS: supports above kLargeSupport (four offers per lane, larger lists).  CF:
// the construction weights are summed over the whole vocabulary (relative to
// the row maximum): for bf16 from counts of the row's values, taken as it
// streams (V = 128256, 256 rows: 32 us a level where a pass of its own for the
// totals took 91 us before the 23 us of the row kernel; 30 now); for fp32, whose
// values hardly repeat, and for rows the counts do not cover, in a second
// pass over the row.
// ---------------------------------------------------------------------------
template <int DT, bool LS, int NTB, bool CF>
__global__ __launch_bounds__(NTB, 4) void k_expand_row(RowArgs) {
    constexpr int VEC = DT ? 8 : 4;
    constexpr int NW = NTB / WAVE;
    constexpr bool COUNT = CF && DT == 1;
    const RowArgs& args = kernel_params<RowArgs>();
    const TreeDev& t = args.t;
    const LevelArgs& a = args.a;
    extern __shared__ __align__(16) uint8_t s_pdyn[];
    __shared__ RowShared<NTB> rs;
    __shared__ PoolShared<NTB> ps;
    __shared__ uint64_t s_wsum[NW], s_wcount[NW];

    ieee_mode_off();                             // NaN words drop out of the maxima
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int row = blockIdx.x;
    const int V = t.V;
    const int NB = row_batches<DT, NTB>(V);
    const RowLds L = row_lds(t.S, LS, NB, NTB, COUNT ? COUNT_ROW : COUNT_NONE);
    uint64_t* s_top = (uint64_t*)(s_pdyn + L.p.top);
    uint8_t* s_tab = s_pdyn + L.tab;
    uint32_t* s_small = (uint32_t*)(s_pdyn + L.small);
    const RowReader<DT, NTB> rd = row_reader<DT, NTB>(t, a, row);
    const RowTop rt = row_top<DT, LS, NTB, COUNT ? COUNT_ROW : COUNT_NONE>(t, a, row, t.S, s_pdyn, L,
                                                                           rd, rs);
    if (COUNT) {
        // the row's total construction weight from the counts of its values;
        // s_wcount checks them: every element of every batch in the tables (no
        // overflow), no value of 2^9 or more, and none at or below -2^9 unless
        // its weight is 0
        uint64_t w = 0, n = 0;
        const uint64_t w0 = cweight(0.0f, rt.vmax, a.k1);
        const uint32_t* tab = (const uint32_t*)s_tab;
        for (int i = tid; i < HIST_WORDS; i += NTB) {
            const uint32_t c0 = tab[i], c1v = tab[HIST_WORDS + i];
            const uint32_t pos = (c0 & 0xFFFFu) + (c1v & 0xFFFFu), neg = (c0 >> 16) + (c1v >> 16);
            n += pos + neg;
            if (i >= 1 && i < HIST_OUT) {
                const float l = hist_value(i);
                w += (uint64_t)pos * cweight(l, rt.vmax, a.k1) + (uint64_t)neg * cweight(-l, rt.vmax, a.k1);
            } else if (i == 0) {
                w += (uint64_t)(pos + neg) * w0;     // (the listed ones put right below)
            } else {
                if (pos != 0 || (neg != 0 && cweight(-512.0f, rt.vmax, a.k1) != 0u)) n += 1ull << 40;
            }
        }
        const int ns = rs.nsmall;
        if (ns > HIST_SMALL) n += 1ull << 40;
        for (int i = tid; i < min(ns, HIST_SMALL); i += NTB)
            w += cweight(__uint_as_float(s_small[i] << 16), rt.vmax, a.k1) - w0;
        w = wave_sum_u64(w);
        n = wave_sum_u64(n);
        if (lane == 0) {
            s_wsum[wid] = w;
            s_wcount[wid] = n;
        }
    }

    if (CF) {
        __syncthreads();
        uint64_t n = 0, w = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            n += COUNT ? s_wcount[q] : 0ull;
            w += COUNT ? s_wsum[q] : 0ull;
        }
        if (!COUNT || n != (uint64_t)(NB * NTB) * (EBATCH * VEC)) {
            const float M = key_value(s_top[0]);
            w = 0;
            for (int bt = 0; bt < NB; ++bt) {
                uint4 r[EBATCH];
                rd.load_batch(r, bt);
#pragma unroll
                for (int e = 0; e < EBATCH; ++e) {
                    // (padding reads as -inf or a NaN word: no weight)
                    const int e0 = rd.vidx(bt * EBATCH + e) * VEC;
#pragma unroll
                    for (int k = 0; k < VEC; ++k) {
                        const uint32_t x = cweight_below(elem<DT>(r[e], k), M, a.k1);
                        w += (e0 + k < V) ? x : 0u;
                    }
                }
            }
            w = wave_sum_u64(w);
            __syncthreads();                     // (s_wsum is read)
            if (lane == 0) s_wsum[wid] = w;
            __syncthreads();
            w = 0;
#pragma unroll
            for (int q = 0; q < NW; ++q) w += s_wsum[q];
        }
        if (tid == 0) ps.s1full = w;             // (read past pool_form's first barrier)
    }
    constexpr int SC = LS ? SMAX : kLargeSupport;    // the largest support of the class
    pool_form<NTB, (SC + NTB - 1) / NTB>(t, a, row, s_pdyn, L.p, rs.pu, rt.pr, rs.u, ps);
    select_frontier(t, a, row / a.P, row % a.P, rt.pr, s_top, (uint64_t*)(s_pdyn + L.p.k2), ps);
}

// Four blocks per CU keep enough loads in flight; the largest chunk variant
// holds twice the registers and runs at two.
template <int DT, int NVC>
__global__ __launch_bounds__(NTC) void k_select(TreeDev t, LevelArgs a) {
    select_block<DT, NVC>(t, a);
}
template <int DT>
__global__ __launch_bounds__(NTC) void k_select_wide(TreeDev t, LevelArgs a) {
    select_block<DT, 32>(t, a);
}

// 16-byte vectors per thread of k_expand; a chunk is NTC * NVC vectors.
static const int kNVC[] = {4, 8, 16, 32};

int expand_variant_count(int) { return (int)(sizeof(kNVC) / sizeof(kNVC[0])); }

ExpandVariant expand_variant(int dtype, int v, int V, int S) {
    const int chunk = NTC * kNVC[v] * (dtype ? 8 : 4);
    ExpandVariant ev;
    ev.chunk = chunk;
    ev.C = (V + chunk - 1) / chunk;
    ev.Sc = S < chunk ? S : chunk;
    ev.ok = (int64_t)ev.C * ev.Sc <= MERGE_MAX;
    return ev;
}

template <int DT>
static void launch_dt(const TreeDev& t, const LevelArgs& a, int v, dim3 grid, size_t shm,
                      hipStream_t s) {
    switch (v) {
    case 0: k_select<DT, 4><<<grid, NTC, shm, s>>>(t, a); break;
    case 1: k_select<DT, 8><<<grid, NTC, shm, s>>>(t, a); break;
    case 2: k_select<DT, 16><<<grid, NTC, shm, s>>>(t, a); break;
    default: k_select_wide<DT><<<grid, NTC, shm, s>>>(t, a); break;
    }
}

hipError_t launch_select(const TreeDev& t, const LevelArgs& a, int variant, hipStream_t s) {
    const int rows = t.B * a.P;
    const dim3 grid(t.C, rows);
    if (t.dtype) launch_dt<1>(t, a, variant, grid, 0, s);
    else launch_dt<0>(t, a, variant, grid, 0, s);
    return hipGetLastError();
}

hipError_t launch_expand(const TreeDev& t, const LevelArgs& a, int variant, hipStream_t s) {
    hipError_t e = launch_select(t, a, variant, s);
    if (e != hipSuccess) return e;
    const size_t shm = (size_t)pool_lds(t.S, t.C).bytes;
    k_pool<<<t.B * a.P, NTP, shm, s>>>(t, a);
    return hipGetLastError();
}

int expand_variant_nvc(int v) { return kNVC[v]; }

// ---------------------------------------------------------------------------
// k_row_wsum: for the whole-vocabulary construction of a sparse tree, the
// total construction weight of every row of the level, sum over all V of
// w(l; M, k1) with M the row maximum (the same weights the pool computes
// on its support).  One block per row, two passes over the row: the
// maximum, then the weights.
// ---------------------------------------------------------------------------
constexpr int NTW = 256;

template <int DT>
__global__ __launch_bounds__(NTW) void k_row_wsum(TreeDev t, LevelArgs a) {
    constexpr int VEC = DT ? 8 : 4;
    __shared__ float s_max[NTW / WAVE];
    __shared__ uint64_t s_sum[NTW / WAVE];
    const int row = blockIdx.x;
    const int V = t.V;
    const int NVR = (V + VEC - 1) / VEC;
    const char* base = (const char*)a.logits + (int64_t)row * t.stride * (DT ? 2 : 4);
    float mx = -INFINITY;
    for (int vi = threadIdx.x; vi < NVR; vi += NTW) {
        const uint4 x = load_row_vec<DT>(base, vi, V);
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (vi * VEC + k < V) mx = fmaxf(mx, elem<DT>(x, k));
    }
    const float M = block_max<NTW>(mx, s_max);
    uint64_t sum = 0;
    for (int vi = threadIdx.x; vi < NVR; vi += NTW) {
        const uint4 x = load_row_vec<DT>(base, vi, V);
#pragma unroll
        for (int k = 0; k < VEC; ++k)
            if (vi * VEC + k < V) sum += cweight(elem<DT>(x, k), M, a.k1);
    }
    sum = block_sum_u64<NTW>(sum, s_sum);
    if (threadIdx.x == 0) t.s1row[row] = sum;
}

hipError_t launch_row_wsum(const TreeDev& t, const LevelArgs& a, hipStream_t s) {
    const dim3 grid(t.B * a.P);
    if (t.dtype) k_row_wsum<1><<<grid, NTW, 0, s>>>(t, a);
    else k_row_wsum<0><<<grid, NTW, 0, s>>>(t, a);
    return hipGetLastError();
}

static size_t row_shm(int dtype, int V, int S, int ntb, bool cfull) {
    const int nvr = (V + (dtype ? 8 : 4) - 1) / (dtype ? 8 : 4);
    const int nb = (nvr + ntb * EBATCH - 1) / (ntb * EBATCH);
    return (size_t)row_lds(S, S > kLargeSupport, nb, ntb,
                           cfull && dtype == 1 ? COUNT_ROW : COUNT_NONE).p.bytes;
}

// Threads of a k_expand_row block for a row of V elements: 512 (64 vectors
// each: 262,144 bf16 or 131,072 fp32 elements), or 1024 for the fp32 rows
// beyond; 0 if the row is too long for either or its LDS does not fit.
int expand_row_threads(int dtype, int V, int S, bool cfull) {
    const int nvr = (V + (dtype ? 8 : 4) - 1) / (dtype ? 8 : 4);
    for (int ntb : {NTE, 2 * NTE})
        if (nvr <= ntb * EBATCH * ROW_BATCHES)
            return row_shm(dtype, V, S, ntb, cfull) <= kRowLdsMax ? ntb : 0;
    return 0;
}

template <int DT, bool CF>
static const void* row_fn(int S, int ntb) {
    // (no bf16 row needs 1024 threads)
    if (ntb == 2 * NTE) {
        if constexpr (DT == 0)
            return S > kLargeSupport ? (const void*)&k_expand_row<DT, true, 2 * NTE, CF>
                                     : (const void*)&k_expand_row<DT, false, 2 * NTE, CF>;
        return nullptr;
    }
    if (S > kLargeSupport) return (const void*)&k_expand_row<DT, true, NTE, CF>;
    return ntb == NTE ? (const void*)&k_expand_row<DT, false, NTE, CF>
                      : (const void*)&k_expand_row<DT, false, NTE / 2, CF>;
}
static const void* row_fn(const TreeDev& t, int ntb) {
    if (t.cfull) return t.dtype ? row_fn<1, true>(t.S, ntb) : row_fn<0, true>(t.S, ntb);
    return t.dtype ? row_fn<1, false>(t.S, ntb) : row_fn<0, false>(t.S, ntb);
}

// A level of more rows than the device holds 512-thread blocks at once
// runs 256-thread blocks, of which it holds more (rows of up to 64 vectors
// per thread, supports of up to 256): the rows past the first round no
// longer wait for a whole block to end.
static bool row_narrow(const TreeDev& t, int rows) {
    const int nvr = (t.V + (t.dtype ? 8 : 4) - 1) / (t.dtype ? 8 : 4);
    if (nvr > NTE / 2 * EBATCH * ROW_BATCHES || t.S > kLargeSupport) return false;
    if (t.row_narrow >= 0) return t.row_narrow == 1;
    return t.row_slots > 0 && rows > t.row_slots;
}

// How many 512-thread blocks of this tree's row kernel the device holds at
// once (0 when the rows are too long for them); raises the kernels' limit on
// dynamic LDS.
hipError_t expand_row_slots(const TreeDev& t, int* slots) {
    *slots = 0;
    int dev = 0, cus = 0, per = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int wide = t.dense ? 0 : expand_row_threads(t.dtype, t.V, t.S, t.cfull != 0);
    for (int ntb : {NTE / 2, wide}) {
        if (e != hipSuccess || wide == 0) break;
        if (ntb == NTE / 2 && (t.S > kLargeSupport || wide != NTE)) continue;
        e = hipFuncSetAttribute(row_fn(t, ntb), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kRowLdsMax);
        if (e == hipSuccess && ntb == NTE) {
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, row_fn(t, ntb), ntb,
                                                             row_shm(t.dtype, t.V, t.S, ntb, t.cfull != 0));
            if (e == hipSuccess) *slots = per * cus;
        }
    }
    return e;
}

hipError_t launch_expand_row(const TreeDev& t, const LevelArgs& a, hipStream_t s) {
    const int rows = t.B * a.P;
    const int ntb = row_narrow(t, rows) ? NTE / 2 : expand_row_threads(t.dtype, t.V, t.S, t.cfull != 0);
    if (ntb == 0) return hipErrorInvalidValue;
    RowArgs ra{t, a};
    ra.a.cached = level_cached(t, t.B * a.P);
    void* args[] = {&ra};
    return hipLaunchKernel(row_fn(t, ntb), dim3(rows), dim3(ntb), args, row_shm(t.dtype, t.V, t.S, ntb, t.cfull != 0), s);
}

}  // namespace rheo
