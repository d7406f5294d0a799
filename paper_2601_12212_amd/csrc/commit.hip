// Input update after verification: the K/V rows of the accepted path (root .. deepest accepted
// node) are appended to every layer's prefix cache; rejected tree tokens are simply never copied.
// One workgroup per (sequence, layer, K or V): at most DT_D_MAX + 1 rows of Hkv * D elements each,
// moved in 16-byte pieces when the layout allows it.  The new prefix length (= position of the next
// root, the bonus token) and the next root token are written by the workgroups of layer 0.
#include "common.hpp"
#include "kernels.hpp"

namespace dt {

typedef u32 Piece __attribute__((ext_vector_type(4)));
// A thread keeps its place u in the row (head g, piece c) and takes every `step`-th row, all of them requested before the
// first is stored (store by store, each row was a trip to memory of its own, behind two integer divisions: 4.6 us for two
// sequences and 32 layers, 3.8 now).
template <typename T>
__device__ __forceinline__ void copy_rows(const CommitArgs &a, const T *tree, T *cache, int L, int rows, const int *node,
                                          int per_head /* units of T per head */) {
    // the cache strides are given in elements, T holds `epu` of them
    const int epu = sizeof(T) / (a.dtype == DT_BF16 ? 2 : 4);
    const int64_t stok = a.kv_stride_tok / epu, shead = a.kv_stride_head / epu;
    const int per_row = a.Hkv * per_head, tid = threadIdx.x;
    const int step = max(256 / per_row, 1);  // rows side by side
    const int s0 = per_row < 256 ? (int)((u32)tid / (u32)per_row) : 0;
    if (s0 >= step) return;
    constexpr int B = 5;  // rows in flight
    for (int u = tid - s0 * per_row; u < per_row; u += 256) {
        const int g = (int)((u32)u / (u32)per_head);
        const T *src = tree + u;
        T *dst = cache + (int64_t)L * stok + (int64_t)g * shead + (u - g * per_head);
        for (int s = s0; s < rows; s += B * step) {
            T v[B];
#pragma unroll
            for (int r = 0; r < B; ++r) v[r] = src[(int64_t)node[min(s + r * step, rows - 1)] * per_row];
#pragma unroll
            for (int r = 0; r < B; ++r)
                if (s + r * step < rows) dst[(int64_t)(s + r * step) * stok] = v[r];
        }
    }
}

__global__ __launch_bounds__(256) void commit_kernel(CommitArgs a) {
    const int b = blockIdx.x, layer = blockIdx.y, kv = blockIdx.z, tid = threadIdx.x;
    __shared__ int s_node[DT_D_MAX + 1];
    // one trip for all the words (path entries past the path are not used)
    const int slot = b * (DT_D_MAX + 1) + min(tid, DT_D_MAX);
    const int my_node = a.path_nodes[slot];
    int n_raw = a.n_nodes[b], len_raw = a.accept_len[b], cap_raw = a.prefix_cap[b], l_raw = a.prefix_len[b];
    const void *tree = (kv ? a.v_tree : a.k_tree)[layer];
    void *cache = (kv ? a.v_prefix : a.k_prefix)[(int64_t)layer * a.batch + b];
    const bool tells = layer == 0 && kv == 0;
    const int my_out = tells && a.next_root_token ? a.out_tokens[slot] : 0;
    // here, all at once (left alone, the words are read one behind the other, where they are first used)
    asm volatile("" : "+s"(n_raw), "+s"(len_raw), "+s"(cap_raw), "+s"(l_raw), "+s"(tree), "+s"(cache));
    const int N = min(max(n_raw, 1), a.TT_cap);
    const int len = min(max(len_raw, 0), DT_D_MAX);
    const int cap = max(cap_raw, 0);
    const int L = min(max(l_raw, 0), cap);
    const int rows = min(len + 1, cap - L);  // rows that still fit
    if (tid <= DT_D_MAX)  // a node index outside the tree (bad input) is clamped, never followed
        s_node[tid] = min(max(my_node, 0), N - 1);
    __syncthreads();
    if (tells) {
        if (tid == 0) a.new_prefix_len[b] = L + rows;
        if (tid == len && a.next_root_token) a.next_root_token[b] = my_out;
    }
    if (rows <= 0) return;
    const int esz = a.dtype == DT_BF16 ? 2 : 4;
    const int64_t tree_seq = (int64_t)b * a.TT_cap * a.Hkv * a.D;  // elements before this sequence's tree rows
    const char *tp = (const char *)tree + tree_seq * esz;
    const bool vec = a.vec16 && ((uintptr_t)tp % 16 == 0) && ((uintptr_t)cache % 16 == 0);
    if (vec) copy_rows<Piece>(a, (const Piece *)tp, (Piece *)cache, L, rows, s_node, a.D * esz / 16);
    else if (esz == 2) copy_rows<uint16_t>(a, (const uint16_t *)tp, (uint16_t *)cache, L, rows, s_node, a.D);
    else copy_rows<uint32_t>(a, (const uint32_t *)tp, (uint32_t *)cache, L, rows, s_node, a.D);
}

hipError_t commit_launch(const CommitArgs &a, hipStream_t st) {
    if (a.batch <= 0 || a.n_layers <= 0) return hipSuccess;
    launch_kernel(KID_COMMIT, st, commit_kernel, dim3(a.batch, a.n_layers, 2), dim3(256), 0, a);
    return hipGetLastError();
}

}  // namespace dt
