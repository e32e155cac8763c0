// Global pruning of the tree (Sec. 2.1; App. C.1): the R best non-root nodes
// by (path score desc, depth asc, slot path asc), their pruned order, and
// what the pruned view and the tree mask read (parent's pruned index, token,
// depth).  Scores never grow along a path (Lemma 2) and the tie-break ranks a
// parent before its children, so the kept set is ancestor-closed; every kept
// node is checked for it.
//
// One 512-thread block per sequence.  Only the nodes near the R-th best are
// compared: the scores are counted in bins of an eighth of an octave (a
// monotone map of the score's high bits), one prefix sum gives every bin's
// first rank, and the exact order inside the bins that begin below rank R
// comes from comparing a bin's members with each other.  The kernel is a
// chain of latencies (one read of the scores, one of the candidates'
// records).  Counting every node against every other, on sixteen blocks a
// sequence, took 6.6 us at 456 nodes and 64 sequences and 21 us at 710 nodes
// and 128; this takes 5.2 and 8.2 us.
#include "rheo_device.h"
#include "rheo_state.h"

namespace rheo {

constexpr int NTR = 512;
constexpr int PBINS = 512;                   // one bin per thread

// The bin of a score in [0, 1] or infinite (score_order): its exponent and three mantissa bits, from 511
// (1 and above) down to 2^-63 and below (0).
__device__ __forceinline__ int score_bin(double s) {
    const int k = (int)((uint64_t)__double_as_longlong(s) >> 49);
    return min(max(k - ((0x3FF << 3) - (PBINS - 1)), 0), PBINS - 1);
}

struct PruneLds {
    int lo, ord, bs, rank, bytes;            // scores first
};
__host__ __device__ inline PruneLds prune_lds(int n) {
    PruneLds L;
    L.lo = 8 * n;
    L.bs = L.lo + 8 * n;
    L.ord = L.bs + 4 * n;
    L.rank = L.ord + 2 * n;
    L.bytes = L.rank + 2 * n;
    return L;
}

__global__ __launch_bounds__(NTR) void k_prune(TreeDev t, int R) {
    extern __shared__ __align__(16) uint8_t s_dyn[];
    __shared__ int s_hist[PBINS], s_start[PBINS];
    __shared__ int s_w[NTR / WAVE];
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % WAVE, wid = tid / WAVE;
    const int n = t.NN - 1;                  // non-root nodes, uids 1..NN-1
    const int64_t nb = (int64_t)b * t.NN;
    const PruneLds L = prune_lds(n);
    double* s_score = (double*)s_dyn;
    uint64_t* s_lo = (uint64_t*)(s_dyn + L.lo);
    int* s_bs = (int*)(s_dyn + L.bs);
    int16_t* s_ord = (int16_t*)(s_dyn + L.ord);
    int16_t* s_rank = (int16_t*)(s_dyn + L.rank);
    s_hist[tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += NTR) {
        const double sc = score_order(t.score[nb + 1 + i]);
        const int bin = score_bin(sc);
        s_score[i] = sc;
        s_bs[i] = bin | (atomicAdd(&s_hist[bin], 1) << 16);
    }
    if (tid == 0) {
        t.node[nb].pidx = 0;
        t.pr_par[nb] = -1;
        t.pr_tok[nb] = -1;
        t.pr_depth[nb] = 0;
    }
    __syncthreads();
    {
        const int v = s_hist[PBINS - 1 - tid];
        int ex = wave_excl_scan(v);
        if (lane == WAVE - 1) s_w[wid] = ex + v;
        __syncthreads();
        for (int w = 0; w < wid; ++w) ex += s_w[w];
        s_start[PBINS - 1 - tid] = ex;
    }
    __syncthreads();
    // candidates: the members of the bins that begin below rank R, with the
    // lower half of their priority key
    for (int i = tid; i < n; i += NTR) {
        const int bs = s_bs[i], st = s_start[bs & 0xFFFF];
        if (st < R) {
            const Node& nd = t.node[nb + 1 + i];
            uint64_t hi, lo;
            prio_key(s_score[i], nd.meta & 0xFF, nd.path, hi, lo);
            s_lo[i] = lo;
            s_ord[st + (bs >> 16)] = (int16_t)i;
        }
    }
    __syncthreads();
    for (int i = tid; i < n; i += NTR) {
        const int bin = s_bs[i] & 0xFFFF, st = s_start[bin];
        int rk = n;
        if (st < R) {
            const double sc = s_score[i];
            const uint64_t lo = s_lo[i];
            rk = st;
            for (int q = st; q < st + s_hist[bin]; ++q) {
                const int o = s_ord[q];
                const double so = s_score[o];
                rk += (int)(so > sc) | ((int)(so == sc) & (int)(s_lo[o] > lo));
            }
        }
        s_rank[i] = (int16_t)(rk < R ? rk + 1 : -1);
        t.node[nb + 1 + i].pidx = rk < R ? rk + 1 : -1;
    }
    __syncthreads();
    for (int i = tid; i < n; i += NTR) {
        const int k = s_rank[i];
        if (k < 0) continue;
        const Node& nd = t.node[nb + 1 + i];
        const int p = nd.par;
        const int pk = p == 0 ? 0 : (p > 0 && p <= n) ? s_rank[p - 1] : -1;
        // a parent outranks its child (raises the sticky error flag if not)
        if (pk < 0 || pk >= k) atomicOr(t.err, 2);
        t.pr_par[nb + k] = pk;
        t.pr_tok[nb + k] = nd.tok;
        t.pr_depth[nb + k] = nd.meta & 0xFF;
    }
}

// Raises the kernel's limit on dynamic LDS to what the largest tree takes (the
// limit is the kernel's, not one tree's).
hipError_t prepare_prune(const TreeDev&) {
    return hipFuncSetAttribute((const void*)&k_prune, hipFuncAttributeMaxDynamicSharedMemorySize,
                               prune_lds(kMaxNodes).bytes);
}

hipError_t launch_prune(const TreeDev& t, int R, hipStream_t s) {
    k_prune<<<t.B, NTR, (size_t)prune_lds(t.NN - 1).bytes, s>>>(t, R);
    return hipGetLastError();
}

}  // namespace rheo
