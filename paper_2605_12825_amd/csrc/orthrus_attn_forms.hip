// The 32-row attention kernel's forms for few rows and for mixed lengths: the body of attn_split_kernel with another compute wave
// or another order of the items.
//
// A code object of their own.  Among the split and merge kernels, whose code they left as it was, they made a batch-1 step
// slower by where its kernels came to lie (sampled step of 4096 tokens, two attention calls and the consensus, 64 rows: 44.0 ->
// 44.3 and 44.9 -> 45.2 us with them among those, 44.7 -> 44.6 and 45.2 -> 45.0 apart).
#include "orthrus_attn_dev.h"

namespace orthrus {

// The compute wave of a call with at most 16 query rows per KV head (a short block, few query heads a KV head, one token at a
// time): v_mfma_f32_16x16x32_bf16 instead of a 32-row block that is half padding.  Same problem, tile layout, masks and
// softmax order; a lane owns row lane % 16, and the four lanes of a row hold a quarter of a tile's scores each.
// What it saves is a wave's chain (8 exponentials a tile for 16, products of 16 cycles for 32: a workgroup with a CU to itself
// takes 0.36 us a tile where a 32-row block takes 0.45), power, and half of every partial: written in the same register order,
// rows 16..31 of a block left out.  32-row block -> this form, us per call (32/8 heads, K = 4, unless said otherwise): one
// sequence of 4096 / 12000 / 40000 tokens 10.5 -> 9.4 / 15.2 -> 14.0 / 28.9 -> 28.5, 36-layer graph of 4096 tokens 835 -> 778
// (the kernel alone 7.85 -> 6.92); 64 of 100 tokens 6.8 -> 6.1; balanced, 17 of 797..12753 91.8 -> 82.0, 64 of 300..3000 92.3 ->
// 82.2; 4 x 40000 103.8 -> 103.0; d = 64, 4 of 12000, 16 rows 12.5 -> 11.4; masks of 2 x 2000, 256 blocks of 8 (16/8 heads) 145 ->
// 102, half of it by their order.  In blocks of 16 for more rows (two waves for 32 rows, four for 64) it reads the tiles
// twice: 10.3 -> 10.0 and 12.0 -> 12.3 at 4096 tokens, a 12-layer graph at batch 2 377 -> 385.
template <int D, int NS, int MODE, int NT>
__device__ __forceinline__ void thin_rows(const AttnArgs &a, WorkItems<MODE> it, uint32_t smem_lds)
{
    using Gm = AttnGeom<D>;
    constexpr int CH = Gm::CH, ROWB = Gm::ROWB, RPI = Gm::RPI, GS = Gm::GS, TILE_B = Gm::TILE_B, STAGE_B = Gm::STAGE_B;
    constexpr int KST = D / 32, NB = D / 16;  // steps along d for the scores, 16-wide output blocks
    constexpr bool BALANCED = MODE == kItemsBalanced;
    const int lane = threadIdx.x & 63, col = lane & 15, quad = lane >> 4;
    const int K = a.block_k, G = a.group;
    int kb[KST];     // K operand: row `col` (+16), chunks 4 * step + quad
    int vb[NB / 2];  // V operand through the transpose read: row 4 * quad + col / 4 (+16)
    {
        const int r = col % RPI;
#pragma unroll
        for (int q = 0; q < KST; ++q) kb[q] = (col / RPI) * GS + r * ROWB + ((q ^ (xm<CH>(r) >> 2)) << 6) + (quad << 4);
        const int tok = 4 * quad + (col >> 2), rv = tok % RPI;
#pragma unroll
        for (int db = 0; db < NB / 2; ++db)
            vb[db] = TILE_B + (tok / RPI) * GS + rv * ROWB + ((db ^ (xm<CH>(rv) >> 2)) << 6) + (((lane & 3) >> 1) << 4) + ((lane & 1) << 3);
    }
    const float c = a.scale_log2e;
    const bool row_ok = col < a.rows;
    const int irow = row_ok ? col / G : 31, hl = col - irow * G;  // (padding rows see every in-block key and are never stored)
    for (;;) {  // one pass per work item (balanced partition: per segment)
        Frag qf[KST];
#pragma unroll
        for (int kk = 0; kk < KST; ++kk) qf[kk].u = make_uint4(0, 0, 0, 0);
        if (row_ok) {
            const uint16_t *qp = a.q + ((int64_t)it.b * K + irow) * a.q_stride_row + ((int64_t)it.g * G + hl) * a.q_stride_head;
#pragma unroll
            for (int kk = 0; kk < KST; ++kk) qf[kk].u = *(const uint4 *)(qp + kk * 32 + quad * 8);
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the queries are in registers before the loop starts
        f32x4 o[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m_run = kNegBig, l_run = 0.f;
        int stage = 0;
        for (int i = 0; i < it.n_tiles; ++i) {
            wg_barrier();
            const uint32_t st = smem_lds + (uint32_t)stage * STAGE_B;
            stage = stage + 1 == NS ? 0 : stage + 1;
            // number of leading tile tokens this lane's row may see
            int lim;
            if (i < it.n_cache) lim = it.t_end - (it.t_begin + i * 32);
            else lim = a.view == 0 ? K : min(K, irow + 1);
            Frag kf[KST][2], vf[NB];  // every operand read goes out before the first product
#pragma unroll
            for (int kk = 0; kk < KST; ++kk)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    kf[kk][t].n = *(const lds_u32x4 *)(uintptr_t)(st + kb[kk] + t * (16 / RPI) * GS);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    vf[nb].h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_s16x4 *)(uintptr_t)(st + vb[nb >> 1] + ((nb & 1) << 5) + t * (16 / RPI) * GS));
            __builtin_amdgcn_sched_barrier(0);
            f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int kk = 0; kk < KST; ++kk)
#pragma unroll
                for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kk][t].v, qf[kk].v, s[t], 0, 0, 0);
            if (lim < 32) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if (16 * (r >> 2) + 4 * quad + (r & 3) >= lim) s[r >> 2][r & 3] = -INFINITY;
            }
            float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
            for (int r = 1; r < 4; ++r) mx = fmaxf(mx, fmaxf(s[0][r], s[1][r]));
            const float m_cand = fmaxf(m_run, max_with_other_half(max_with_other_row(mx)) * c);
            if (__any(m_cand - m_run > kLazy)) {
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_cand);
                m_run = m_cand;
                l_run *= alpha;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) o[nb] *= alpha;
            }
            float p[8], sum = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r >> 2][r & 3], c, -m_run));
                sum += p[r];
            }
            l_run += sum;
            // the product's k-slot (quad, j) is token 16 * (j / 4) + 4 * quad + j % 4, on either side
            Frag pf;
            pf.u = make_uint4(pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7]));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) o[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[nb].v, pf.v, o[nb], 0, 0, 0);
        }
        l_run = sum_with_other_half(sum_with_other_row(l_run));
        if (it.final_out) {
            const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
            // lanes of even and odd quads trade eights of two blocks, as the 32-row form's halves do (store_row)
            uint16_t *op = a.out + (((int64_t)it.b * K + irow) * a.num_q_heads + (int64_t)it.g * G + hl) * D + (quad & 1) * 12 + quad * 4;
#pragma unroll
            for (int nb = 0; nb < NB; nb += 2) {
                const auto x = __builtin_amdgcn_permlane16_swap(pack_bf16(o[nb][0] * inv, o[nb][1] * inv),
                                                                pack_bf16(o[nb + 1][0] * inv, o[nb + 1][1] * inv), false, false);
                const auto y = __builtin_amdgcn_permlane16_swap(pack_bf16(o[nb][2] * inv, o[nb][3] * inv),
                                                                pack_bf16(o[nb + 1][2] * inv, o[nb + 1][3] * inv), false, false);
                if (row_ok) *(uint4 *)(op + nb * 16) = make_uint4(x[0], y[0], x[1], y[1]);
            }
            if (a.lse && quad == 0 && row_ok)
                a.lse[((int64_t)it.b * a.num_q_heads + (int64_t)it.g * G + hl) * K + irow] =
                    (m_run + __builtin_amdgcn_logf(l_run)) * 0.6931471805599453f;
        } else if (row_ok) {
            f32x4 *po = (f32x4 *)a.part_o + it.part_slot * (D / 32 * 4 * 64) + (quad >> 1) * 64 + (quad & 1) * 32 + col;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (NT == 1 && !BALANCED) __builtin_nontemporal_store(o[nb], &po[nb * 128]);
                else po[nb * 128] = o[nb];
            }
            if (quad == 0) ((float2 *)a.part_ml)[it.part_slot * 32 + col] = make_float2(m_run, l_run);
        }
        if (!BALANCED || !it.open(a)) break;
        wg_barrier();  // matches the loader's barrier between segments
    }
}

// Fixed splits, the long items first.  A kernel of its own: the search for a workgroup's item in front of a batch-1 call's
// code cost that call 0.3 % (36-layer graph 940 -> 943 us), though it never ran.
template <int D, int W, int NS, int NT>
__global__ void __launch_bounds__(64 * (W + 1), 3) attn_by_size_kernel(ATTN_FIRST_PARAMS, const AttnArgs rest)
{
    constexpr int MODE = kItemsBySize, PROBE = 0, ROWS = 32;
#include "orthrus_attn_split.inc"
}

// At most 16 query rows per KV head (thin_rows).
template <int D, int NS, int MODE, int NT>
__global__ void __launch_bounds__(128, 3) attn_thin_kernel(ATTN_FIRST_PARAMS, const AttnArgs rest)
{
    constexpr int W = 1, PROBE = 0, ROWS = 16;
#include "orthrus_attn_split.inc"
}

template <int D>
static auto thin_kernel(const AttnPlan &plan)
{
    if (plan.bal_wgs > 0) return attn_thin_kernel<D, kStages, kItemsBalanced, kNtAsked>;
    if (plan.by_size) return plan.kv_nt ? attn_thin_kernel<D, kStages, kItemsBySize, 1> : attn_thin_kernel<D, kStages, kItemsBySize, 0>;
    return plan.kv_nt ? attn_thin_kernel<D, kStages, kItemsSplit, 1> : attn_thin_kernel<D, kStages, kItemsSplit, 0>;
}

hipError_t launch_attn_thin(const AttnArgs &a, const AttnPlan &plan, int head_dim, dim3 grid, hipStream_t stream, AttnLaunchEvents *ev)
{
    auto kern = head_dim == 128 ? thin_kernel<128>(plan) : thin_kernel<64>(plan);
    return launch_timed(kern, grid, dim3(128), plan.lds_bytes, a, stream, ev, 0);
}

template <int D, int W>
static auto by_size_kernel(int nt) { return nt ? attn_by_size_kernel<D, W, kStages, 1> : attn_by_size_kernel<D, W, kStages, 0>; }

template <int D>
static auto by_size_kernel(const AttnPlan &plan)
{
    switch (plan.waves) {
    case 1: return by_size_kernel<D, 1>(plan.kv_nt);
    case 2: return by_size_kernel<D, 2>(plan.kv_nt);
    case 3: return by_size_kernel<D, 3>(plan.kv_nt);
    case 4: return by_size_kernel<D, 4>(plan.kv_nt);
    case 5: return by_size_kernel<D, 5>(plan.kv_nt);
    case 6: return by_size_kernel<D, 6>(plan.kv_nt);
    case 7: return by_size_kernel<D, 7>(plan.kv_nt);
    default: return by_size_kernel<D, 8>(plan.kv_nt);
    }
}

hipError_t launch_attn_by_size(const AttnArgs &a, const AttnPlan &plan, int head_dim, dim3 grid, hipStream_t stream, AttnLaunchEvents *ev)
{
    auto kern = head_dim == 128 ? by_size_kernel<128>(plan) : by_size_kernel<64>(plan);
    return launch_timed(kern, grid, dim3(64 * (plan.waves + 1)), plan.lds_bytes, a, stream, ev, 0);
}

}  // namespace orthrus
