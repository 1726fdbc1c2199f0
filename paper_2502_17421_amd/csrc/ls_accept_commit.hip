// The two integer steps that follow the attention in a verification round: greedy acceptance
// of the speculation tree (Section 3.3 "Fast Tree Attention", evaluated at T = 0 in Section
// 4.1) and the move of the accepted tokens' key/value rows into the cache (the cache is
// updated only once verification is complete, Section 3.2; "KV cache movement" in the
// appendix "Experiments Details").  Both are latency-bound: a tree has at most LS_MAX_TREE nodes.
#include "ls_internal.hpp"

namespace ls {

namespace {

// One workgroup per sequence; a thread takes nodes tid, tid + blockDim.x, ...
//   match[i]    node i carries the token the target predicts after its parent
//   child_of[p] the lowest matching child of p (lowest index wins among equal tokens)
// The accepted path starts at node 0 and follows child_of until a node has no matching child;
// children come after their parents, so the walk ends after at most n_tree steps.
//
// Bound by latency: one round trip for the three token arrays, two LDS passes, and the walk, one
// LDS read per accepted node.  Siblings compete with an LDS minimum per parent; the form before
// compared every matching node with all earlier ones and let every node walk up to the root, one
// LDS read after the other (128 nodes, 4 sequences: 12.9 us, this form 2.4 us).
__global__ void __launch_bounds__(256)
tree_accept_kernel(const int32_t *__restrict__ parents, const int32_t *__restrict__ draft,
                   const int32_t *__restrict__ target, int32_t n_tree, int32_t *__restrict__ path,
                   int32_t *__restrict__ accept_len, int32_t *__restrict__ next_token,
                   int32_t *__restrict__ err_flag)
{
    constexpr int NPT = LS_MAX_TREE / 256;  // nodes per thread, for the smallest workgroup that may see LS_MAX_TREE nodes
    __shared__ int32_t tgt[LS_MAX_TREE];
    __shared__ int32_t child_of[LS_MAX_TREE];
    __shared__ int32_t path_sh[LS_MAX_TREE];
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int step = blockDim.x;  // n_tree <= NPT * step
    parents += (size_t)b * n_tree;
    draft += (size_t)b * n_tree;
    target += (size_t)b * n_tree;
    path += (size_t)b * n_tree;

    int bad = 0;
    int32_t par[NPT], own[NPT];
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int i = tid + k * step;
        par[k] = -1;
        own[k] = 0;
        if (i >= n_tree) continue;
        par[k] = parents[i];
        own[k] = draft[i];
        tgt[i] = target[i];
        child_of[i] = LS_MAX_TREE;
        path_sh[i] = -1;
        if (par[k] < -1 || par[k] >= i) {  // not a forest in topological order: treat the node as a root
            bad = 1;
            par[k] = -1;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NPT; ++k)
        if (par[k] >= 0 && own[k] == tgt[par[k]]) atomicMin(&child_of[par[k]], tid + k * step);
    const int any_bad = __syncthreads_or(bad);
    if (tid == 0) {
        int cur = 0, len = 0;
        while (true) {
            path_sh[len++] = cur;
            const int next = child_of[cur];
            if (next >= n_tree) break;
            cur = next;
        }
        next_token[b] = tgt[cur];  // the token the target adds itself after the deepest accepted node
        accept_len[b] = len;
        if (err_flag) err_flag[b] = any_bad ? 1 : 0;
    }
    __syncthreads();
    for (int i = tid; i < n_tree; i += step) path[i] = path_sh[i];
}

// One workgroup per (sequence, KV head): 16-byte pieces of the accepted rows of K and V are
// copied from the tree buffers to cache rows prefix_len, prefix_len + 1, ...  The number of
// rows moved is the longest prefix of the path whose entries are nodes and whose target rows
// exist; anything shorter than accept_len is reported in err_flag.
//
// Bound by latency as well: lengths and path, then the rows, then the stores.
__global__ void __launch_bounds__(256)
kv_commit_kernel(Problem p, int elem_bytes, const int32_t *__restrict__ accept_path,
                 const int32_t *__restrict__ accept_len, uint8_t *__restrict__ k_cache,
                 uint8_t *__restrict__ v_cache, int32_t *__restrict__ new_prefix_lens,
                 int32_t *__restrict__ err_flag)
{
    __shared__ int32_t path[LS_MAX_TREE];
    __shared__ int32_t n_sh;
    const int b = blockIdx.x / p.n_kv_heads;
    const int g = blockIdx.x % p.n_kv_heads;
    const int tid = threadIdx.x;

    // the whole path, together with the lengths that say how much of it counts: one round trip
    constexpr int NPT = LS_MAX_TREE / 256;
    int32_t node[NPT];
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int t = tid + k * 256;
        node[k] = t < p.n_tree ? accept_path[(size_t)b * p.n_tree + t] : -1;
    }
    int plen = p.prefix_lens[b];
    plen = plen < 0 ? 0 : (plen > p.max_prefix_len ? p.max_prefix_len : plen);
    int want = accept_len[b];
    want = want < 0 ? 0 : (want > p.n_tree ? p.n_tree : want);
    int room = p.max_prefix_len - plen;
    int n = want < room ? want : room;
    if (tid == 0) n_sh = n;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int t = tid + k * 256;
        if (t >= n) continue;
        path[t] = node[k];
        if (node[k] < 0 || node[k] >= p.n_tree) atomicMin(&n_sh, t);  // stop before the first bad entry
    }
    __syncthreads();
    n = n_sh;

    // 16-byte pieces per row: 8, 16 or 32 (head_dim 64 or 128, elements of 2 or 4 bytes)
    const int chunk_shift = __builtin_ctz((uint32_t)(p.head_dim * elem_bytes / 16));
    const uint8_t *kt = (const uint8_t *)p.k_tree + (b * p.kt_stride[0] + g * p.kt_stride[1]) * elem_bytes;
    const uint8_t *vt = (const uint8_t *)p.v_tree + (b * p.vt_stride[0] + g * p.vt_stride[1]) * elem_bytes;
    // contiguous cache: first index = sequence; paged cache: first index = page, found per row
    const int32_t *tab = p.block_table ? p.block_table + (size_t)b * p.bt_stride : nullptr;
    const int page_rows_mask = (1 << p.page_shift) - 1;
    for (int e = tid; e < n << chunk_shift; e += blockDim.x) {
        const int j = e >> chunk_shift, c = e & ((1 << chunk_shift) - 1);
        const int64_t node = path[j];
        const int row = plen + j;  // < max_prefix_len <= bt_stride * page size
        const int64_t first = tab ? (int64_t)tab[row >> p.page_shift] : (int64_t)b;
        const int64_t in_row = tab ? (row & page_rows_mask) : row;
        const uint4 kv = *(const uint4 *)(kt + node * p.kt_stride[2] * elem_bytes + c * 16);
        const uint4 vv = *(const uint4 *)(vt + node * p.vt_stride[2] * elem_bytes + c * 16);
        *(uint4 *)(k_cache + (first * p.kc_stride[0] + g * p.kc_stride[1] + in_row * p.kc_stride[2]) * elem_bytes +
                   c * 16) = kv;
        *(uint4 *)(v_cache + (first * p.vc_stride[0] + g * p.vc_stride[1] + in_row * p.vc_stride[2]) * elem_bytes +
                   c * 16) = vv;
    }
    if (g == 0 && tid == 0) {
        if (new_prefix_lens) new_prefix_lens[b] = plen + n;
        if (err_flag) err_flag[b] = n < accept_len[b] ? 1 : 0;
    }
}

}  // namespace

hipError_t launch_tree_accept(const int32_t *parents, const int32_t *draft_tokens, const int32_t *target_tokens,
                              int32_t batch, int32_t n_tree, int32_t *accept_path, int32_t *accept_len,
                              int32_t *next_token, int32_t *err_flag, hipStream_t stream)
{
    const int threads = n_tree <= 64 ? 64 : (n_tree <= 128 ? 128 : 256);
    hipLaunchKernelGGL(tree_accept_kernel, dim3(batch), dim3(threads), 0, stream, parents, draft_tokens,
                       target_tokens, n_tree, accept_path, accept_len, next_token, err_flag);
    return hipGetLastError();
}

hipError_t launch_kv_commit(const Problem &p, int dtype, const int32_t *accept_path, const int32_t *accept_len,
                            void *k_cache, void *v_cache, int32_t *new_prefix_lens, int32_t *err_flag,
                            hipStream_t stream)
{
    const int elem_bytes = is_16bit(dtype) ? 2 : 4;
    hipLaunchKernelGGL(kv_commit_kernel, dim3(p.batch * p.n_kv_heads), dim3(256), 0, stream, p, elem_bytes,
                       accept_path, accept_len, (uint8_t *)k_cache, (uint8_t *)v_cache, new_prefix_lens, err_flag);
    return hipGetLastError();
}

}  // namespace ls
