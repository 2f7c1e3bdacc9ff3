// Verification hand-off (Method, "Inference": the draft tree is verified in
// one pass with an equality check; Experiments, "Metrics": block efficiency
// counts the accepted tokens plus the verifier's residual token).
//
// tree_inputs_kernel lays a draft tree out for a verifier pass with tree
// attention: position 0 is the root token, position 1 + j node j (pop
// order); positions are depths; mask[i][j] = 1 when position j is position i
// or one of its ancestors.  accept_kernel walks the tree with the verifier's
// next token at every position: from the root, to the child carrying the
// current position's target, while there is one.
#include "common.hpp"
#include "launch.hpp"

namespace tf {

constexpr int kVerifyThreads = 256;
constexpr int kMaskRows = 32;   // positions a workgroup lays out

// Workgroup (sequence, 32 positions).  What bounds it is dependent steps, and
// for large trees the mask's stores (263 KB a sequence at 512 nodes), which one
// workgroup a sequence pushed through one CU; rows are independent, so
// they are dealt out: 512 nodes, one sequence 5.9 -> 2.8 us, sixteen 7.1 -> 3.6;
// 16 x 32 nodes 2.5 both ways, about a launch.
// Parents are staged in LDS; a node's parent must precede it (pop order), which
// also bounds every ancestor walk and the parents a workgroup needs.
__global__ __launch_bounds__(kVerifyThreads) void tree_inputs_kernel(const int32_t* __restrict__ root_token,
                                                                     const int32_t* __restrict__ node_token,
                                                                     const int32_t* __restrict__ node_parent,
                                                                     const int32_t* __restrict__ node_depth, int B,
                                                                     int32_t* __restrict__ tokens,
                                                                     int32_t* __restrict__ positions,
                                                                     uint8_t* __restrict__ mask) {
    extern __shared__ int32_t par[];
    const int s = blockIdx.x;
    const int tid = threadIdx.x;
    const int n = B + 1;
    const int i0 = blockIdx.y * kMaskRows, i1 = min(i0 + kMaskRows, n);   // positions [i0, i1)
    const int32_t* tk = node_token + (size_t)s * B;
    const int32_t* pa = node_parent + (size_t)s * B;
    const int32_t* dp = node_depth + (size_t)s * B;
    int32_t* to = tokens + (size_t)s * n;
    int32_t* po = positions + (size_t)s * n;
    uint8_t* m = mask + ((size_t)s * n + i0) * n;

    for (int j = tid; j < i1 - 1; j += kVerifyThreads) par[j] = pa[j];
    const int i = i0 + tid;
    if (i < i1) {
        to[i] = i == 0 ? root_token[s] : tk[i - 1];
        po[i] = i == 0 ? 0 : dp[i - 1];
    }
    // zero the rows: 16-byte stores on the aligned middle, bytes at the ends
    const size_t total = (size_t)(i1 - i0) * n;
    const size_t head = (16 - (reinterpret_cast<uintptr_t>(m) & 15)) & 15;
    const size_t h = head < total ? head : total;
    for (size_t e = tid; e < h; e += kVerifyThreads) m[e] = 0;
    const size_t nvec = (total - h) / 16;
    uint4* mv = reinterpret_cast<uint4*>(m + h);
    for (size_t e = tid; e < nvec; e += kVerifyThreads) mv[e] = uint4{0u, 0u, 0u, 0u};
    for (size_t e = h + nvec * 16 + tid; e < total; e += kVerifyThreads) m[e] = 0;
    __syncthreads();   // zeros stored and parents staged before the ones below

    if (i < i1) {
        uint8_t* row = m + (size_t)tid * n;
        row[0] = 1;
        if (i > 0) {
            row[i] = 1;
            int child = i - 1;
            int p = par[child];
            while (p >= 0 && p < child) {   // ancestors in pop order always precede
                row[1 + p] = 1;
                child = p;
                p = par[p];
            }
        }
    }
}

// One workgroup per sequence.  Every node looks at once whether the verifier
// picked it at its parent, and the first such child of a position is kept in
// LDS, so the walk is a chain of single LDS reads instead of a search of all
// nodes and a load of the target at every step (three or four accepted: 16
// sequences of 32 nodes 3.3 -> 2.4 us, of 512 5.9 -> 2.8).
__global__ __launch_bounds__(kVerifyThreads) void accept_kernel(const int32_t* __restrict__ node_token,
                                                                const int32_t* __restrict__ node_parent,
                                                                const int32_t* __restrict__ target, int B,
                                                                int max_depth, int32_t* __restrict__ accepted,
                                                                int32_t* __restrict__ accept_len,
                                                                int32_t* __restrict__ bonus) {
    extern __shared__ int32_t next[];   // [B + 1]: first child with the position's target, B: none
    __shared__ int s_len;
    const int s = blockIdx.x;
    const int tid = threadIdx.x, nth = blockDim.x;
    const int32_t* tk = node_token + (size_t)s * B;
    const int32_t* pa = node_parent + (size_t)s * B;
    const int32_t* tg = target + (size_t)s * (B + 1);
    int32_t* acc = accepted + (size_t)s * max_depth;
    for (int i = tid; i <= B; i += nth) next[i] = B;
    __syncthreads();
    for (int j = tid; j < B; j += nth) {
        const int p = pa[j], t = tk[j];
        if (p >= -1 && p < B && tg[1 + p] == t) atomicMin(&next[1 + p], j);
    }
    __syncthreads();
    if (tid == 0) {
        int cur = -1, len = 0;
        while (len < max_depth) {
            const int hit = next[1 + cur];
            if (hit >= B) break;
            acc[len] = hit;
            cur = hit;
            ++len;
        }
        s_len = len;
        accept_len[s] = len;
        bonus[s] = tg[1 + cur];
    }
    __syncthreads();
    for (int i = s_len + tid; i < max_depth; i += nth) acc[i] = -1;
}

hipError_t launch_tree_inputs(const int32_t* root_token, const int32_t* node_token, const int32_t* node_parent,
                              const int32_t* node_depth, int b, int B, int32_t* tokens, int32_t* positions,
                              uint8_t* mask, hipStream_t stream) {
    hipLaunchKernelGGL(tree_inputs_kernel, dim3(b, (B + kMaskRows) / kMaskRows), dim3(kVerifyThreads),
                       (size_t)B * 4, stream, root_token, node_token, node_parent, node_depth, B, tokens, positions, mask);
    return hipGetLastError();
}

hipError_t launch_accept(const int32_t* node_token, const int32_t* node_parent, const int32_t* target, int b, int B,
                         int max_depth, int32_t* accepted, int32_t* accept_len, int32_t* bonus, hipStream_t stream) {
    // a wave holds a small tree's nodes (and keeps millions of sequences within a grid's 2^32 threads)
    const int threads = B <= 64 || b >= (1 << 23) ? 64 : kVerifyThreads;
    hipLaunchKernelGGL(accept_kernel, dim3(b), dim3(threads), (size_t)(B + 1) * 4, stream, node_token, node_parent,
                       target, B, max_depth, accepted, accept_len, bonus);
    return hipGetLastError();
}

}  // namespace tf
