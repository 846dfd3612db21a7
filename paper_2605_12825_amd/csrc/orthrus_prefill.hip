// Front end of the AR view's prefill (Section 3.1: the frozen AR view processes the context with its
// ordinary causal self-attention and leaves its K/V in the cache that both views share afterwards).
//
//   prefill_append_kernel  grid (token block, sequence): every workgroup validates its sequence's lengths and
//                          that every page the new tokens fall on is mapped (the same answer everywhere), then
//                          copies its 16 new tokens' K/V rows into their pages with 16-byte accesses.  The first
//                          one records the length before the call and the accepted number of new tokens (0 after
//                          an error) for the attention, whose first chunk bumps seq_lens: nothing here may,
//                          while others still read it.
// (A planning launch in front of the copy cost 5 us of every call, and the copy, one load and store at a time, 16 us
// for 8192 tokens of 8 heads.)
// The attention itself is the prefill form of attn_wide_kernel, or of attn_split_kernel for small launches
// (prefill_wide_waves in orthrus_attn_wide.hip).
#include "orthrus_internal.h"

namespace orthrus {

constexpr int kAppendRows = 16;  // new tokens per workgroup

__global__ void __launch_bounds__(256) prefill_append_kernel(const PrefillArgs a)
{
    const int b = blockIdx.y, i0 = blockIdx.x * kAppendRows, tid = threadIdx.x;
    const int L = a.seq_lens[b];
    int n = a.new_lens_in[b];
    bool bad = L < 0 || n < 0 || n > a.max_new || (int64_t)L + n > a.max_seq_len;
    if (!bad) {
        // pages of positions L .. L+n-1
        const int first = L >> a.page_shift, last = n > 0 ? (L + n - 1) >> a.page_shift : first - 1;
        for (int slot = first + tid; slot <= last; slot += 256) {
            if (slot >= a.max_pages_per_seq) bad = true;
            else {
                const int pg = a.page_table[(int64_t)b * a.max_pages_per_seq + slot];
                if (pg < 0 || pg >= a.num_pages) bad = true;
            }
        }
    }
    const bool any_bad = __syncthreads_or(bad);
    if (any_bad) n = 0;
    if (blockIdx.x == 0 && tid == 0) {
        if (any_bad) atomicExch(a.err_word, -4);
        a.old_lens[b] = L < 0 ? 0 : L;
        a.new_lens[b] = n;
    }
    if (i0 >= n) return;
    const int rows = min(kAppendRows, n - i0);
    const int H = a.num_kv_heads, d = a.head_dim;
    const int cpr = d / 8;  // 16-byte chunks per row
    const int per_tok = H * cpr;
    const int P = 1 << a.page_shift;
    // the rows of new tokens are contiguous, so chunk e of the block sits at e * 8; four chunks of K and V per thread
    // are loaded before the first is stored
    const int64_t src0 = ((int64_t)b * a.max_new + i0) * per_tok * 8;
    const int total = rows * per_tok;
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    for (int e0 = tid; e0 < total; e0 += 4 * 256) {
        u32x4 k[4], v[4];
        int64_t dst[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = min(e0 + u * 256, total - 1);  // (past the end: the last chunk again, not stored)
            const int t = e / per_tok, rem = e - t * per_tok;
            const int g = rem / cpr, ch = rem - g * cpr;
            const int pos = L + i0 + t;
            const int pg = a.page_table[(int64_t)b * a.max_pages_per_seq + (pos >> a.page_shift)];
            dst[u] = (int64_t)pg * a.stride_page + (int64_t)g * a.stride_head + (int64_t)(pos & (P - 1)) * a.stride_tok + ch * 8;
            k[u] = *(const u32x4 *)(a.k_new + src0 + (int64_t)e * 8);
            v[u] = *(const u32x4 *)(a.v_new + src0 + (int64_t)e * 8);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (e0 + u * 256 < total) {
                *(u32x4 *)(a.k_pool + dst[u]) = k[u];
                *(u32x4 *)(a.v_pool + dst[u]) = v[u];
            }
    }
}

hipError_t launch_prefill_append(const PrefillArgs &a, hipStream_t stream)
{
    if (a.batch == 0) return hipSuccess;
    if (a.max_new == 0) return hipSuccess;
    dim3 grid((unsigned)((a.max_new + kAppendRows - 1) / kAppendRows), (unsigned)a.batch);
    hipLaunchKernelGGL(prefill_append_kernel, grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace orthrus
