// Small copy-out kernels for the ABI's view calls.
#include "rheo_device.h"
#include "rheo_state.h"

namespace rheo {

__global__ void k_read_nodes(TreeDev t, int32_t* token, int32_t* parent, int32_t* depth,
                             int32_t* slot, int32_t* kind, double* proxy, double* qtrue,
                             double* score) {
    const int64_t n = (int64_t)t.B * t.NN;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int meta = t.node[i].meta;
        if (token) token[i] = t.node[i].tok;
        if (parent) parent[i] = t.node[i].par;
        if (depth) depth[i] = meta & 0xFF;
        if (slot) slot[i] = (meta >> 8) & 0xFF;
        if (kind) kind[i] = (meta >> 16) & 0xFF;
        if (proxy) proxy[i] = t.node[i].proxy;
        if (qtrue) qtrue[i] = t.node[i].qtrue;
        if (score) score[i] = t.node[i].score;
    }
}

__global__ void k_pruned_view(TreeDev t, int R, int32_t* parent, int32_t* token) {
    const int64_t n = (int64_t)t.B * (R + 1);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int b = (int)(i / (R + 1));
        const int64_t o = (int64_t)b * t.NN + (i - (int64_t)b * (R + 1));
        if (parent) parent[i] = t.pr_par[o];
        if (token) token[i] = t.pr_tok[o];
    }
}

// The mask and the depths of one sequence, by `split` blocks: the parents'
// pruned indices in LDS, one ancestor walk (at most depth <= 15 steps, to
// ever smaller indices; where the error flag says that a parent was pruned,
// to -1 or not at all) per entry.
constexpr int NTM = 256;

__global__ __launch_bounds__(NTM) void k_tree_mask(TreeDev t, int R, int split,
                                                   uint8_t* mask, int32_t* depth) {
    extern __shared__ int s_par[];
    const int n = R + 1;
    const int b = blockIdx.x / split, part = blockIdx.x % split;
    const int64_t nb = (int64_t)b * t.NN;
    for (int i = threadIdx.x; i < n; i += NTM) {
        s_par[i] = min(max(t.pr_par[nb + i], -1), R);
        if (depth && part == 0) depth[(int64_t)b * n + i] = t.pr_depth[nb + i];
    }
    __syncthreads();
    if (!mask) return;
    uint8_t* out = mask + (int64_t)b * n * n;
    for (int e = part * NTM + threadIdx.x; e < n * n; e += NTM * split) {
        const int i = e / n, j = e - i * n;
        int p = i;
        for (int s = 0; s < 16 && p > j; ++s) p = s_par[p];
        out[e] = (p == j) ? 1 : 0;
    }
}

hipError_t launch_tree_mask(const TreeDev& t, int R, uint8_t* mask, int32_t* depth,
                            hipStream_t s) {
    // Blocks of a sequence: four entries a thread, so that one large mask fills
    // the chip (one sequence, R = 400: 5.1 us with sixteen entries a thread, 145 us
    // at R = 1000 by four blocks), at least four and at most 8192 in all, beyond
    // which each would only read the parents again (32 sequences, R = 3000: 242 us).
    const int64_t n2 = (int64_t)(R + 1) * (R + 1);
    int64_t split = (n2 + 4 * NTM - 1) / (4 * NTM);
    if (split > 8192 / t.B) split = 8192 / t.B;
    if (split < 4) split = 4;
    k_tree_mask<<<t.B * (int)split, NTM, sizeof(int) * (size_t)(R + 1), s>>>(t, R, (int)split, mask,
                                                                         depth);
    return hipGetLastError();
}

hipError_t launch_read_nodes(const TreeDev& t, int32_t* token, int32_t* parent,
                             int32_t* depth, int32_t* slot, int32_t* kind, double* proxy,
                             double* qtrue, double* score, hipStream_t s) {
    const int64_t n = (int64_t)t.B * t.NN;
    const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    k_read_nodes<<<blocks, 256, 0, s>>>(t, token, parent, depth, slot, kind, proxy, qtrue,
                                        score);
    return hipGetLastError();
}

hipError_t launch_pruned_view(const TreeDev& t, int R, int32_t* parent, int32_t* token,
                              hipStream_t s) {
    const int64_t n = (int64_t)t.B * (R + 1);
    const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    k_pruned_view<<<blocks, 256, 0, s>>>(t, R, parent, token);
    return hipGetLastError();
}

}  // namespace rheo
