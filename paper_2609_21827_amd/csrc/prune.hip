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
// comes from comparing a bin's members with each other, which lie side by
// side in LDS and are read eight at a time.  The kernel is a chain of
// latencies (one read of the scores, one of the candidates' records).
// Counting every node against every other, on sixteen blocks a sequence, took
// 6.6 us at 392 nodes and 64 sequences and 22.5 us at 710 nodes and 128; this
// takes 4.3 and 6.9 us.
//
// A bin of many members costs their number squared, so the bins follow where
// scores pile up: scores of 0 (weights of 0 below confident rows) have a bin
// per depth, which is their next criterion; trees of more nodes than threads,
// whose deep scores pass below the 62 octaves of the other bins (flat rows:
// eleven octaves a level at V = 2048), take coarser ones if their least score
// needs them.  3165 nodes of equal rows, R = 3000: 111 us by counting all, 460
// with the scores below 2^-63 in one bin, 59 so.
#include "rheo_device.h"
#include "rheo_state.h"

namespace rheo {

constexpr int NTR = 512;
constexpr int PBINS = 512;                   // one bin per thread
constexpr int ZBINS = 15;                    // of them, for scores of 0: one per depth
constexpr int kOne = 0x3FF << 3;             // score_bits of 1

// The exponent of a score and three bits of its mantissa.
__device__ __forceinline__ int score_bits(double s) {
    return (int)((uint64_t)__double_as_longlong(s) >> 49);
}
// The bin of a score in [0, 1] or infinite (score_order), of a node of
// index i among the non-root nodes: 511 for 1 and above.
__device__ __forceinline__ int score_bin(double s, int coarse, const TreeDev& t, int i) {
    if (s == 0.0) {
        const int above = i < t.K ? 0 : 1 + (i - t.K) / (t.NE * t.K);   // depth - 1
        return ZBINS - 1 - above;
    }
    return min(max(((score_bits(s) - kOne) >> coarse) + PBINS - 1, ZBINS), PBINS - 1);
}

struct alignas(16) ScoreKey {
    double score;
    uint64_t lo;                             // lower half of the priority key
};
constexpr int KSTEP = 8;                     // keys compared at a time

struct PruneLds {
    int score, bs, rank, bytes;              // the keys, in bin order, first
};
__host__ __device__ inline PruneLds prune_lds(int n) {
    PruneLds L;
    L.score = 16 * (n + KSTEP);
    L.bs = L.score + 8 * n;
    L.rank = L.bs + 4 * n;
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
    ScoreKey* s_key = (ScoreKey*)s_dyn;
    double* s_score = (double*)(s_dyn + L.score);
    int* s_bs = (int*)(s_dyn + L.bs);
    int16_t* s_rank = (int16_t*)(s_dyn + L.rank);
    s_hist[tid] = 0;
    int coarse = 0;
    int least = kOne;
    for (int i = tid; i < n; i += NTR) {
        const double sc = score_order(t.score[nb + 1 + i]);
        s_score[i] = sc;
        if (sc != 0.0) least = min(least, score_bits(sc));
    }
    if (n > NTR) {
        // the widest bins whose range does not end above the least score
        for (int o = 1; o < WAVE; o <<= 1) least = min(least, __shfl_xor(least, o));
        if (lane == 0) s_w[wid] = least;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NTR / WAVE; ++w) least = min(least, s_w[w]);
        while (((kOne - least) >> coarse) > PBINS - 1 - ZBINS) ++coarse;
    }
    __syncthreads();
    for (int i = tid; i < n; i += NTR) {
        const int bin = score_bin(s_score[i], coarse, t, i);
        s_bs[i] = bin | (atomicAdd(&s_hist[bin], 1) << 16);
    }
    if (tid < KSTEP) s_key[n + tid].score = -1.0;
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
    // every score in bin order, and for the candidates, the members of the bins
    // that begin below rank R, the lower half of their priority key
    for (int i = tid; i < n; i += NTR) {
        const int bs = s_bs[i], st = s_start[bs & 0xFFFF];
        ScoreKey& k = s_key[st + (bs >> 16)];
        k.score = s_score[i];
        k.lo = 0;                            // (ranks below every candidate of its score)
        if (st < R) {
            const Node& nd = t.node[nb + 1 + i];
            uint64_t hi;
            prio_key(k.score, nd.meta & 0xFF, nd.path, hi, k.lo);
        }
    }
    __syncthreads();
    for (int i = tid; i < n; i += NTR) {
        const int bin = s_bs[i] & 0xFFFF, st = s_start[bin];
        int rk = n;
        if (st < R) {
            const ScoreKey me = s_key[st + (s_bs[i] >> 16)];
            rk = st;
            // (keys past the bin rank lower and count for nothing)
            for (int q = st; q < st + s_hist[bin]; q += KSTEP) {
                ScoreKey k[KSTEP];
#pragma unroll
                for (int u = 0; u < KSTEP; ++u) k[u] = s_key[q + u];
#pragma unroll
                for (int u = 0; u < KSTEP; ++u)
                    rk += (int)(k[u].score > me.score) |
                          ((int)(k[u].score == me.score) & (int)(k[u].lo > me.lo));
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
