// The attention kernel for launches that are bound by arithmetic: prefill, and decode-mode batches with enough query
// rows and units to fill the chip (the training block mask above all).  Same problem, MFMA forms, LDS tile layout
// and masks as attn_split_kernel, never split along the keys (orthrus_attn.hip); what differs is how a CU is filled.
//
// Why: with 32 query rows per wave every 32-token tile costs a wave 16 KB of LDS reads for 512 cycles of matrix
// instructions, and a wave's own chain (operand reads, scores, softmax, values) leaves the matrix cores idle for most
// of it: 37 % busy in an 8192-token prefill with two such waves on each SIMD.  Here a wave owns 64 rows as two blocks
// (one wave per SIMD, up to 512 registers), so an operand read serves two products, and the two blocks are half a tile
// apart: while block 0's scores of tile i and values of tile i-1 go through the matrix cores, the vector unit takes
// block 1's softmax of tile i-1, and the other way round in the second half ("slots").  Inside a slot every matrix
// instruction is followed by its share of the softmax and of the LDS reads and loads, in written order
// (sched_barrier): the compiler's own order keeps them apart.
// Every wave issues its own share of the tile loads (a loader wave would halve the registers), NS-1 tiles ahead.
//
// What bounds it: issue, and at full load the power that the products draw.  One wave issues a vector instruction every
// 6 to 8 cycles, other ones every 4, so whatever is not a product or softmax costs time: a product with its share of the
// softmax (multiply-add, exponential, sum, half a conversion) takes 35 cycles against the product's own 32, and the rest
// of a tile's instructions come on top.  The main loop therefore takes a turn of the ring at a time, so that LDS
// addresses are instruction offsets, waits for LDS twice a tile, and keeps the memory addresses of 64 tiles in vector
// registers: 190 instructions a 64x32 tile (counters: 157 vector ones with the products, 24 LDS, 5 scalar, 4 loads) where an
// address calculation and a wait at each use made it 225.  Measured before and after: one item to a CU (100 new tokens
// behind 16000, 7 heads a KV head) 351 -> 291 us a call; 16384 new tokens (32/8 heads) 1763 -> 1670, where the kernel's cycles
// fall by 13 %, the products' share of them rises from 0.61 to 0.70 and the clock falls from 1.97 to 1.81 GHz; 8192 new tokens
// 478 -> 456; ragged prefill at 28/4 heads 325 -> 300; training mask 623 -> 598.  (attn_split_kernel's form: 675, 400 and 864
// for the last three.  With the chunks ranked over all sequences the ragged prefill takes 250 to 280 by the order of the
// lengths, with 16-byte stores the mask 570 to 602 from one card to another.)
#include "orthrus_attn_dev.h"

#include <utility>

namespace orthrus {

template <int... S, class F>
__device__ __forceinline__ void for_each_stage(std::integer_sequence<int, S...>, F &&f)
{
    (f(std::integral_constant<int, S>{}), ...);
}

// D head_dim, W waves of 64 query rows, NS LDS stages, MODE the work items (not kItemsBalanced), NT the
// non-temporal form of the tile loads.
template <int D, int W, int NS, int MODE, int NT = 0>
__global__ void __launch_bounds__(64 * W, 1) attn_wide_kernel(ATTN_FIRST_PARAMS, const AttnArgs rest)
{
    const AttnArgs a = with_first(rest, first_lens, first_batch);
    using Gm = AttnGeom<D>;
    constexpr int CH = Gm::CH, ROWB = Gm::ROWB, RPI = Gm::RPI, NI = Gm::NI, GS = Gm::GS;
    constexpr int TILE_B = Gm::TILE_B, STAGE_B = Gm::STAGE_B, KSTEPS = Gm::KSTEPS, DBLK = Gm::DBLK;
    constexpr int LPW = 2 * NI / W;  // load instructions per tile and wave
    static_assert(2 * NI % W == 0, "the waves share a tile's loads evenly");
    constexpr int PG = 4 / W;  // of a tile's four 16-token halves (K, K, V, V), how many a wave loads
    static_assert(W == 2 || W == 4, "a wave's halves stay within one operand");
    static_assert(NS >= 4 && (NS - 3) * LPW < 64, "stage count");
    static_assert(MODE != kItemsBalanced, "one work item per workgroup");
    constexpr bool PREFILL = MODE == kItemsPrefill;
    using NtTag = std::integral_constant<bool, NT != 0>;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int K = a.block_k, G = a.group;
    const int P = 1 << a.page_shift;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;

    WorkItems<MODE> w;
    w.start(a);
    if (!w.open(a, true)) return;

    // ---- tile loads: a tile is four 16-token halves (K, K, V, V) and a wave loads PG of them, both of one operand
    const int ld_tok = lane / CH;  // this lane's row inside one wave-wide load, and the byte offset of its chunk in that row
    const uint32_t ld_swz = (uint32_t)(((lane % CH) ^ xm<CH>(ld_tok)) << 4);
    HalfLoads<D> half(a, lane);
    const int my_half = wave * PG % 2;
    const bool my_v = wave * PG >= 2;
    const uint32_t my_dst = (my_v ? TILE_B : 0) + my_half * half.GPH * GS;
    const uint32_t dst_first = smem_lds + my_dst, dst_end = dst_first + NS * STAGE_B;
    const uint16_t *my_operand = (my_v ? a.v_pool : a.k_pool) + w.head_off;
    const char *my_pool = half.lowered(my_operand);
    uint32_t worst = 0;  // largest page id that this lane has fetched
    const int n_whole = half.usable ? min(w.n_cache, (w.t_end - w.t_begin) >> 5) : 0;  // tiles loaded a half at a time
    uint32_t dst = dst_first;                                     // where the next tile to be issued goes
    uint32_t page_at = (uint32_t)(w.t_begin + my_half * 16);      // token position of this wave's first half of that tile
    auto advance = [&]() __attribute__((always_inline)) {
        dst = dst + STAGE_B == dst_end ? dst_first : dst + STAGE_B;
        page_at += 32;
    };
    // Where the halves of 64 whole tiles start in memory, a tile to a lane: one vector load and a few vector
    // instructions for 64 tiles, and two lane reads for a half when it is issued.  (A scalar load of the page id and the
    // address arithmetic on it were 24 of the ~105 instructions that a tile costs next to its products and softmax.)
    uint32_t at_lo[PG], at_hi[PG];
    int win = 0;  // tile of lane 0
    auto open_window = [&](int t) __attribute__((always_inline)) {
        win = t;
        const uint32_t tok = (uint32_t)(w.t_begin + min(t + lane, n_whole - 1) * 32 + my_half * 16);
        uint32_t id[PG];
#pragma unroll
        for (int u = 0; u < PG; ++u) id[u] = (uint32_t)((const int32_t *)w.pt_row)[(tok + u * 16u) >> a.page_shift];
        // one wait for all of them: the compiler's wait for an id counts its own loads only, so that one behind a tile
        // load would wait for the tile as well
        if constexpr (PG == 2) asm volatile("" : "+v"(id[0]), "+v"(id[PG - 1]));
#pragma unroll
        for (int u = 0; u < PG; ++u) {
            worst = max(worst, id[u]);
            const uint64_t at = (uint64_t)(uintptr_t)my_pool + (uint64_t)(id[u] < half.num_pages ? id[u] : 0u) * half.page_bytes +
                                ((tok + u * 16u) & half.page_mask) * half.tok_bytes;
            at_lo[u] = (uint32_t)at;
            at_hi[u] = (uint32_t)(at >> 32);
        }
    };
    auto half_base = [&](int u, int t) __attribute__((always_inline)) {
        return (const char *)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)at_lo[u], t - win) |
                              (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)at_hi[u], t - win) << 32);
    };
    // any tile t, outside the main loop
    auto issue_tile = [&](int t) __attribute__((always_inline)) {
        if (t < n_whole) {
            int page[PG];
#pragma unroll
            for (int u = 0; u < PG; ++u) page[u] = w.pt_row[(page_at + u * 16u) >> a.page_shift];
#pragma unroll
            for (int u = 0; u < PG; ++u)
                half.issue(NtTag{}, my_pool + half.offset(page[u], page_at + u * 16u), dst + u * half.GPH * GS);
        } else if (PREFILL || t < w.n_cache) {
            // the last, ragged cache tile: rows past the end repeat the last valid row (finite data, masked later), so
            // nothing is fetched through an unmapped page and no LDS row is left undefined
#pragma unroll 1
            for (int e = 0; e < PG * half.GPH; ++e) {
                const int tg = min((int)page_at + e * RPI + ld_tok, w.t_end - 1);
                const int first = min((int)page_at + e * RPI / 16 * 16, w.t_end - 1);
                const uint32_t id = (uint32_t)w.pt_row[first >> a.page_shift];  // (a load's rows lie in one page)
                half.worst = max(half.worst, id);
                const int64_t off = (int64_t)(id < half.num_pages ? id : 0u) * a.stride_page + (int64_t)(tg & (P - 1)) * a.stride_tok;
                dma16(NtTag{}, my_operand + off + (ld_swz >> 1), dst + e * GS);
            }
        } else {
            // the in-block tile; rows past the block repeat its last row
            const uint16_t *blk = (my_v ? a.v_blk : a.k_blk) + (int64_t)w.b * K * a.blk_stride_row + (int64_t)w.g * a.blk_stride_head;
#pragma unroll 1
            for (int e = 0; e < PG * half.GPH; ++e)
                dma16(NtTag{}, blk + (int64_t)min(my_half * 16 + e * RPI + ld_tok, K - 1) * a.blk_stride_row + (ld_swz >> 1), dst + e * GS);
        }
        advance();
    };

    // ---- lane-invariant LDS read offsets inside one stage
    int kb[KSTEPS / 2];
    {
        const int r = col % RPI;
#pragma unroll
        for (int q = 0; q < KSTEPS / 2; ++q)
            kb[q] = (col / RPI) * GS + r * ROWB + ((q ^ (xm<CH>(r) >> 2)) << 6) + (h << 4);
    }
    int vb[DBLK];
    {
        const int tok0 = 4 * h + ((lane & 15) >> 2);
        const int r = tok0 % RPI;
        const int tr_ch = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
            vb[db] = TILE_B + (tok0 / RPI) * GS + r * ROWB + ((db ^ (xm<CH>(r) >> 2)) << 6) + (tr_ch << 4) + ((lane & 1) << 3);
    }
    const float c = a.scale_log2e;
    // ---- pipeline fill (the page ids of the whole fill in one round trip)
    if (n_whole >= NS - 1) {
        open_window(0);
#pragma unroll
        for (int t = 0; t < NS - 1; ++t) {
#pragma unroll
            for (int u = 0; u < PG; ++u) half.issue(NtTag{}, half_base(u, t), dst + u * half.GPH * GS);
            advance();
        }
    } else {
#pragma unroll 1
        for (int t = 0; t < NS - 1; ++t)
            if (t < w.n_tiles) issue_tile(t);
    }

    // ---- queries: block x holds rows wave*64 + 32*x + col
    Frag qf[2][KSTEPS];
    int irow[2];
    bool row_ok[2];
    const int64_t row_base = PREFILL ? (int64_t)w.b * a.max_new + w.row0 : (int64_t)w.b * K;
    const int rows = w.rows_live * G;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int ridx = wave * 64 + x * 32 + col;
        row_ok[x] = ridx < rows;
        const int i = ridx / G, hl = ridx - i * G;
        irow[x] = row_ok[x] ? i : w.rows_live - 1;
        if (row_ok[x]) {
            const uint16_t *qp = a.q + (row_base + i) * a.q_stride_row + ((int64_t)w.g * G + hl) * a.q_stride_head;
#pragma unroll
            for (int kk = 0; kk < KSTEPS; ++kk) qf[x][kk].u = *(const uint4 *)(qp + kk * 16 + h * 8);
        } else {
#pragma unroll
            for (int kk = 0; kk < KSTEPS; ++kk) qf[x][kk].u = make_uint4(0, 0, 0, 0);
        }
    }
    // tiles of this wave: n_full that every row sees whole, n_mine that any row sees
    int n_full, n_mine;
    if constexpr (PREFILL) {
        const int i0 = wave * 64 / G;
        const int i1 = min((wave * 64 + 63) / G, w.rows_live - 1);
        n_full = i0 < w.rows_live ? (w.pos0 + i0 + 1) >> 5 : 0;
        n_mine = i0 < w.rows_live ? ((w.pos0 + i1) >> 5) + 1 : 0;
    } else {
        n_full = (w.t_end - w.t_begin) >> 5;
        n_mine = w.n_tiles;
    }
    auto limit = [&](int x, int i) __attribute__((always_inline)) -> int {
        if constexpr (PREFILL) return w.pos0 + irow[x] + 1 - i * 32;
        if (i < w.n_cache) return w.t_end - (w.t_begin + i * 32);
        return a.view == 0 ? K : min(K, irow[x] + 1);
    };

    f32x16 o[2][DBLK], s[2];
    float m[2], l[2];
    Frag kf[KSTEPS], vf[DBLK][2], p[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        m[x] = kNegBig;
        l[x] = 0.f;
        p[x][0].u = p[x][1].u = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) s[x][r] = -INFINITY;
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[x][db][r] = 0.f;
    }
    // LDS reads at a stage that is known when the kernel is compiled (S >= 0): the stage is part of the instruction's
    // 16-bit offset, from one of two bases; at any other stage: an add per base.
    constexpr int SPB = 3;  // stages behind one base
    static_assert(NS <= 2 * SPB && SPB * STAGE_B <= 65536, "");
    uint32_t ka[2][KSTEPS / 2], va[2][DBLK];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int q = 0; q < KSTEPS / 2; ++q) {
            ka[u][q] = smem_lds + u * SPB * STAGE_B + kb[q];
            asm("" : "+v"(ka[u][q]));
        }
#pragma unroll
        for (int db = 0; db < DBLK; ++db) {
            va[u][db] = smem_lds + u * SPB * STAGE_B + vb[db];
            asm("" : "+v"(va[u][db]));
        }
    }
    auto read_k = [&](auto stage, uint32_t st, int kk) __attribute__((always_inline)) {
        constexpr int S = decltype(stage)::value;
        uint32_t ad;
        if constexpr (S >= 0) {
            ad = ka[S / SPB][kk >> 1] + S % SPB * STAGE_B;
        } else {
            ad = st + kb[kk >> 1];
            asm("" : "+v"(ad));
        }
        kf[kk].n = *(const lds_u32x4 *)(uintptr_t)(ad + ((kk & 1) << 5));
    };
    auto read_v = [&](auto stage, uint32_t st, int db, int q2) __attribute__((always_inline)) {
        constexpr int S = decltype(stage)::value;
        uint32_t ad;
        if constexpr (S >= 0) {
            ad = va[S / SPB][db] + S % SPB * STAGE_B;
        } else {
            ad = st + vb[db];
            asm("" : "+v"(ad));
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
            vf[db][q2].h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_s16x4 *)(uintptr_t)(ad + (2 * q2 + q) * (8 / RPI) * GS));
    };
    using AnyStage = std::integral_constant<int, -1>;
    constexpr int NCH = KSTEPS + 2 * DBLK;  // products of a slot
    constexpr int VPC = 16 / NCH;           // softmax values handled next to each of them
    // One slot: the matrix work of block C (scores of tile i, values of tile i-1) next to the softmax of the other
    // block's last scores, one product and VPC values at a time.  `extra(j, after)` adds the waits that
    // go in front of product j (after = false) and the loads that go behind it (after = true).
    auto slot = [&](auto cb, auto masked, int lim, auto &&extra) __attribute__((always_inline)) {
        constexpr int C = decltype(cb)::value, X = 1 - C;
        f32x16 z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = 0.f;
        float e[16], sum = 0.f;
        f32x16 t;
        uint32_t pk[8];
        const float mref = m[X];
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            extra(j, std::integral_constant<bool, false>{});
            if (j < KSTEPS) {
                z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j].v, qf[C][j].v, z, 0, 0, 0);
            } else {
                const int db = (j - KSTEPS) % DBLK, q2 = (j - KSTEPS) / DBLK;
                o[C][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][q2].v, p[C][q2].v, o[C][db], 0, 0, 0);
            }
            extra(j, std::integral_constant<bool, true>{});
#pragma unroll
            for (int v = 0; v < VPC; ++v) {
                const int r = j * VPC + v;
                t[r] = s[X][r];
                if constexpr (decltype(masked)::value) {
                    const int tok = 8 * (r >> 2) + 4 * h + (r & 3);
                    t[r] = tok >= lim ? -INFINITY : t[r];
                }
                e[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(t[r], c, -mref));
                if (r == 1) sum = e[0];
                else if (r > 1) sum += e[r - 1];
                if ((r & 1) && r >= 3) pk[(r - 3) / 2] = pack_bf16(e[r - 3], e[r - 2]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        sum += e[15];
        pk[7] = pack_bf16(e[14], e[15]);
        asm volatile("" : "+v"(sum), "+v"(pk[0]), "+v"(pk[1]), "+v"(pk[2]), "+v"(pk[3]), "+v"(pk[4]), "+v"(pk[5]), "+v"(pk[6]), "+v"(pk[7]));
        float alpha;
        if (__builtin_expect(may_outgrow(sum), 0) && move_reference(t, c, m[X], e, sum, alpha)) {
            l[X] *= alpha;
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[X][db][r] *= alpha;
#pragma unroll
            for (int r = 1; r < 16; r += 2) pk[r / 2] = pack_bf16(e[r - 1], e[r]);
        }
        l[X] += sum;
        p[X][0].u = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        p[X][1].u = make_uint4(pk[4], pk[5], pk[6], pk[7]);
        s[C] = z;
    };
    // The barrier inside tile i's step: tile i+1 has landed, the stage of tile i-1 is free and takes tile i+NS-1.
    auto step_barrier = [&](int i) __attribute__((always_inline)) {
        const int ahead = min(NS - 3, w.n_tiles - 2 - i);
        if (ahead >= 3) wait_vmcnt<3 * LPW>();
        else if (ahead == 2) wait_vmcnt<2 * LPW>();
        else if (ahead == 1) wait_vmcnt<LPW>();
        else wait_vmcnt<0>();
        wg_barrier();
        if (i + NS - 1 < w.n_tiles) issue_tile(i + NS - 1);
    };
    // The pipeline's first pass multiplies zero weights, where an infinite V would make NaN of the sums: it reads the V
    // half of the last stage, which holds zeros until the barrier of the first step lets a tile into it.
    const uint32_t last_v = smem_lds + (NS - 1) * STAGE_B + TILE_B;
    for (int x = tid * 16; x < TILE_B; x += 64 * W * 16) *(lds_u32x4 *)(uintptr_t)(last_v + x) = u32x4{0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // tile 0 has landed
    {
        const int ahead = min(NS - 2, w.n_tiles - 1);
        if (ahead >= 3) wait_vmcnt<3 * LPW>();
        else if (ahead == 2) wait_vmcnt<2 * LPW>();
        else if (ahead == 1) wait_vmcnt<LPW>();
        else wait_vmcnt<0>();
        wg_barrier();
    }
    uint32_t st = smem_lds, sv = smem_lds + (NS - 1) * STAGE_B;  // stages of tiles i and i-1
    auto next = [&](uint32_t x) __attribute__((always_inline)) { return x + STAGE_B == smem_lds + NS * STAGE_B ? smem_lds : x + STAGE_B; };
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) read_k(std::integral_constant<int, 0>{}, st, kk);
#pragma unroll
    for (int db = 0; db < DBLK; ++db) vf[db][0].u = make_uint4(0, 0, 0, 0);
    // One tile step.  The reads of a step go out well before their products, in two groups with one wait each (a wait in
    // front of every product costs an issue slot each): next tile's keys as soon as this tile's last product with them is
    // out, the first half of this tile's values (for the next step) behind them, the second half when the next step
    // starts.  S >= 0: the ring stage of tile i, and the step issues the whole tile i+NS-1.
    auto tile = [&](auto stage, auto masked, int i) __attribute__((always_inline)) {
        constexpr int S = decltype(stage)::value;
        constexpr bool FAST = S >= 0;
        using Prev = std::integral_constant<int, FAST ? (S + NS - 1) % NS : -1>;
        using Next = std::integral_constant<int, FAST ? (S + 1) % NS : -1>;
        constexpr int JK = NCH == 16 ? 4 : 2;  // the first read of the next tile's keys
        slot(std::integral_constant<int, 0>{}, masked, limit(1, i - 1), [&](int j, auto after) __attribute__((always_inline)) {
            if constexpr (!decltype(after)::value) {
                if (j == 0) __builtin_amdgcn_s_waitcnt(0xc07f | 2 * DBLK << 8);  // lgkmcnt: all but the values behind the keys
                if (j == KSTEPS) __builtin_amdgcn_s_waitcnt(0xc07f);             // lgkmcnt(0)
            } else if (j < DBLK) {
                read_v(Prev{}, sv, j, 1);
            }
        });
        uint64_t base[PG];
        slot(std::integral_constant<int, 1>{}, masked, limit(0, i), [&](int j, auto after) __attribute__((always_inline)) {
            if constexpr (!decltype(after)::value) return;
            if constexpr (FAST) {
                if (j == 0) {
                    wait_vmcnt<(NS - 3) * LPW>();
                    wg_barrier();
#pragma unroll
                    for (int u = 0; u < PG; ++u) {
                        base[u] = (uint64_t)(uintptr_t)half_base(u, i + NS - 1);
                        asm volatile("" : "+s"(base[u]));
                    }
                }
                // the base was read from a lane two products ago, and nothing passes the scheduling barriers between
                // them, so the load does without its own wait (training mask 593.3 -> 589.7 us, 8192 new tokens
                // 455.6 -> 454.6)
#pragma unroll
                for (int u = 0; u < PG; ++u)
                    if (j == 2 + u)
                        half.template issue<true>(NtTag{}, (const char *)base[u], dst_first + Prev::value * STAGE_B + u * half.GPH * GS);
            } else if (j == 0) {
                step_barrier(i);
                sv = st;
                st = next(st);
            }
            if (j >= JK && j < JK + KSTEPS) read_k(Next{}, st, j - JK);
            if (j >= NCH - DBLK) read_v(stage, sv, j - (NCH - DBLK), 0);
        });
    };
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0): queries and keys are in registers before the loop starts
    int i = 0;
    // steps that issue a whole tile and whose rows see all of theirs, a turn of the ring at a time
    const int n_fast = min(n_full, n_whole - (NS - 1)) / NS * NS;
    while (i < n_fast) {
        if (i + 2 * NS - 2 - win >= 64) open_window(i + NS - 1);
        for_each_stage(std::make_integer_sequence<int, NS>{},
                       [&](auto stage) __attribute__((always_inline)) { tile(stage, std::false_type{}, i + decltype(stage)::value); });
        i += NS;
        page_at += 32 * NS;
    }
    for (; i < n_full; ++i) tile(AnyStage{}, std::false_type{}, i);
    for (; i < n_mine; ++i) tile(AnyStage{}, std::true_type{}, i);
    // drain: the last tile's value products (its second block's softmax in between)
#pragma unroll
    for (int db = 0; db < DBLK; ++db) read_v(AnyStage{}, sv, db, 1);
    slot(std::integral_constant<int, 0>{}, std::true_type{}, limit(1, n_mine - 1), [](int, auto) {});
#pragma unroll
    for (int q2 = 0; q2 < 2; ++q2)
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
            o[1][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][q2].v, p[1][q2].v, o[1][db], 0, 0, 0);
    for (; i < w.n_tiles; ++i) step_barrier(i);

    // ---- write-out (every workgroup holds all of its rows' keys)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float lt = sum_with_other_half(l[x]);
        if (!row_ok[x]) continue;
        const int hl = wave * 64 + x * 32 + col - irow[x] * G;
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        uint16_t *op = a.out + ((row_base + irow[x]) * a.num_q_heads + (int64_t)w.g * G + hl) * D;
        store_row<DBLK>(op, o[x], inv, h);
        if (!PREFILL && a.lse && h == 0)
            a.lse[((int64_t)w.b * a.num_q_heads + (int64_t)w.g * G + hl) * K + irow[x]] =
                (m[x] + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f;
    }
    if (max(worst, half.worst) >= half.num_pages) atomicExch(a.err_word, -4);
}

// ---------------------------------------------------------------------------------------------
// host side

// LDS ring stages: four waves have the CU's LDS to themselves, two workgroups of two waves share it
constexpr int wide_stages(int W) { return W == 4 ? 6 : 4; }

int attn_wide_per_cu(int waves) { return 4 / waves; }  // one wave per SIMD

size_t attn_wide_lds(int waves, int head_dim)
{
    return (size_t)wide_stages(waves) * (head_dim == 128 ? AttnGeom<128>::STAGE_B : AttnGeom<64>::STAGE_B);
}

// Decode mode: whether this kernel beats attn_split_kernel when neither cuts a unit.  It needs waves that are nearly all
// rows (7/8; of 96 rows the training mask takes 626 -> 640 us), units enough for a wave on every SIMD, and lengths over
// which its shorter tile makes up for the longer start and end.  The lines were drawn with the former main loop; both sides
// with today's (attn_split_kernel -> this kernel, us per call, lengths equal to the bound; 256 CUs):
//   d = 128, up to 128 rows: 512 units of 64 / 300 / 1000 tokens at 112 rows 13.6 -> 14.9 / 27.6 -> 27.3 / 64.4 -> 60.8, of
//     180 at 128 rows 21.1 -> 20.6, 896 of 180 40.5 -> 40.9; 256 units of 1000 32.9 -> 36.7; a second round for a few units
//     pays only when it is long or the lengths are mixed, which a long bound suggests (640 units of 400 tokens 45.0 -> 49.8,
//     544 of 1000 79.8 -> 81.5, 640 of 2000 and of 200..1800 1.01 and 1.02 times as fast, the mask's 544 over 1024 / 2048
//     tokens 1.11 and 1.25; 768 units of 400 52.2 -> 54.4)
//   d = 128, more rows: two such waves' work is what four 32-row waves with a loader do as well; 224 rows lose everywhere
//     (1024 units of 1000 tokens 160 -> 164), 256 rows gain from about 2000 tokens on (384 units of 1000 / 2500 tokens
//     76.0 -> 72.2 / 176 -> 144, 256 units of 3000 110 -> 102; masks of 384 over 1024 and of 512 over 2048 tokens 52.4 -> 52.1
//     and 105 -> 97)
//   d = 64, up to 128 rows: 512 units lose at any length (3000 tokens: 83.5 -> 90.1), 640 of 400 / 1000 tokens 22.5 ->
//     22.4 / 48.2 -> 44.6 but the mask's 640 and 704 over 2048 tokens 47.7 -> 52.6 and 52.2 -> 54.7; 768 of 180 / 256 tokens
//     16.1 -> 17.5 / 17.5 -> 18.2, 1024 of 400 38.8 -> 34.3
//   d = 64, more rows: 320 units of 300 / 512 / 1000 tokens at 256 rows 22.1 -> 20.7 / 28.7 -> 25.1 / 48.2 -> 39.0, 256 of
//     700 / 1000 19.9 -> 20.8 / 26.6 -> 25.2; at 224 rows 384 units of 700 / 2000 tokens 29.2 -> 30.5 / 81.6 -> 71.3, the
//     mask's 352 over 4096 tokens 0.96 times as fast, its 384 1.12
// So a few calls now lie on the wrong side: the 32-row kernel keeps 256 rows of d = 128 at 256 units of 3000 (7 %) and 384 of
// 1000 (5 %), and of d = 64 640 units of 1000 at 128 rows (8 %) and 320 of 300 at 256 (6 %); this kernel takes 768 units of
// 400 (4 %), and of d = 64 704 of the mask's (5 %) and 768 of 256 tokens (4 %).
bool attn_wide_pays(int head_dim, int rows, int max_seq_len, int64_t units, int num_cus)
{
    const int waves = rows > 128 ? 4 : 2;
    const int64_t cus = num_cus;
    const bool full = rows >= 60 * waves;
    if (rows < 56 * waves) return false;
    if (waves == 2) {
        if (head_dim == 64) return max_seq_len >= 256 && 4 * units >= 11 * cus;
        if (full && max_seq_len >= 128 && (units == 2 * cus || 2 * units >= 7 * cus)) return true;
        return max_seq_len >= 384 && (units == 2 * cus || units >= 3 * cus || (units > 2 * cus && max_seq_len >= 1024));
    }
    if (head_dim == 128) return full && max_seq_len >= 1920 && units > cus;
    if (!full) return max_seq_len >= 1024 && 2 * units >= 3 * cus;
    return max_seq_len >= 896 ? units >= cus : max_seq_len >= 512 && 4 * units >= 5 * cus;
}

template <int D, int W>
static auto wide_decode_kernel(const AttnPlan &plan)
{
    if (plan.by_size) return plan.kv_nt ? attn_wide_kernel<D, W, wide_stages(W), kItemsBySize, 1> : attn_wide_kernel<D, W, wide_stages(W), kItemsBySize, 0>;
    return plan.kv_nt ? attn_wide_kernel<D, W, wide_stages(W), kItemsSplit, 1> : attn_wide_kernel<D, W, wide_stages(W), kItemsSplit, 0>;
}

hipError_t launch_attn_wide(const AttnArgs &a, const AttnPlan &plan, int head_dim, dim3 grid, hipStream_t stream, AttnLaunchEvents *ev)
{
    auto kern = head_dim == 128 ? (plan.waves == 4 ? wide_decode_kernel<128, 4>(plan) : wide_decode_kernel<128, 2>(plan))
                                : (plan.waves == 4 ? wide_decode_kernel<64, 4>(plan) : wide_decode_kernel<64, 2>(plan));
    return launch_timed(kern, grid, dim3(64 * plan.waves), plan.lds_bytes, a, stream, ev, 0);
}

// Ranked order: a few sequences, and more items than are resident at once.  Items that all start together need no order, and
// finding a rank costs each of them two round trips and the search (plain -> ranked: 16 sequences of 0..2000 cached and up to
// 33 new tokens, 32/8 heads, 44.7 -> 48.8 us with the former search; 8 of 0..3000 and 100..300, 4/2 heads of 64, 48.2 -> 50.0).
bool prefill_ranked(int batch, int64_t items, int per_cu, int num_cus)
{
    return batch > 1 && batch <= kRankedBatch && items > (int64_t)per_cu * num_cus;
}

namespace {
// 64 lanes as arrays: the search above, compiled for the host
struct HostLanes {
    struct Int {
        int v[64];
        Int(int x = 0) { for (int &y : v) y = x; }
        template <class F>
        static Int each(const Int &a, const Int &b, F f) { Int r; for (int i = 0; i < 64; ++i) r.v[i] = f(a.v[i], b.v[i]); return r; }
        friend Int operator+(const Int &a, const Int &b) { return each(a, b, [](int x, int y) { return x + y; }); }
        friend Int operator-(const Int &a, const Int &b) { return each(a, b, [](int x, int y) { return x - y; }); }
        friend Int operator*(const Int &a, const Int &b) { return each(a, b, [](int x, int y) { return x * y; }); }
        friend Int operator>>(const Int &a, int n) { return each(a, n, [](int x, int y) { return x >> y; }); }
    };
    static Int lane() { Int r; for (int i = 0; i < 64; ++i) r.v[i] = i; return r; }
    static Int lesser(const Int &a, const Int &b) { return Int::each(a, b, [](int x, int y) { return x < y ? x : y; }); }
    static Int larger(const Int &a, const Int &b) { return Int::each(a, b, [](int x, int y) { return x > y ? x : y; }); }
    template <class F>
    static Int over_row(const Int &a, F f)
    {
        Int r;
        for (int i = 0; i < 64; ++i) {
            int x = a.v[i & 48];
            for (int j = 1; j < 16; ++j) x = f(x, a.v[(i & 48) + j]);
            r.v[i] = x;
        }
        return r;
    }
    static Int row_sum(const Int &a) { return over_row(a, [](int x, int y) { return x + y; }); }
    static Int row_max(const Int &a) { return over_row(a, [](int x, int y) { return x > y ? x : y; }); }
    static uint64_t less(const Int &a, const Int &b)
    {
        uint64_t m = 0;
        for (int i = 0; i < 64; ++i) m |= (uint64_t)(a.v[i] < b.v[i]) << i;
        return m;
    }
    static int read(const Int &a, int lane) { return a.v[lane]; }
};
}  // namespace

bool ranked_chunk_on_host(int rank, int batch, const int *end_levels, const int *chunks, int *seq, int *chunk)
{
    HostLanes::Int e, n;
    for (int i = 0; i < 64; ++i) {
        const int x = i & 15;
        e.v[i] = x < batch ? end_levels[x] : 0;
        n.v[i] = x < batch ? chunks[x] : 0;
    }
    return ranked_chunk<HostLanes>(rank, e, n, seq, chunk);
}

template <int D, int W>
static hipError_t launch_prefill_wide(AttnArgs a, int num_cus, hipStream_t stream)
{
    a.chunk_tokens = 64 * W / a.group;
    a.rows = 64 * W;
    a.num_splits = (a.max_new + a.chunk_tokens - 1) / a.chunk_tokens;
    dim3 grid((unsigned)a.num_splits * (unsigned)a.num_kv_heads * (unsigned)a.batch);
    a.ranked = prefill_ranked(a.batch, grid.x, attn_wide_per_cu(W), num_cus);
    hipLaunchKernelGGL((attn_wide_kernel<D, W, wide_stages(W), kItemsPrefill>), grid, dim3(64 * W), attn_wide_lds(W, D), stream, ATTN_FIRST_VALUES(a), a);
    return hipGetLastError();
}

// Prefill forms.  A 32-row wave with its own loader is the shorter chain, so for up to four waves a workgroup
// attn_split_kernel's prefill form stays while SIMDs would be idle otherwise.  How long that is depends on how the items'
// lengths are spread (32-row form -> this kernel, us per call):
//   - From 0 up, the new tokens being most of what is cached (by the bound: max_seq_len < 2 * max_new): the longest items
//     start first and short ones fill in behind them.  One sequence of n tokens:
//     d = 128: group 4, 2 heads, n = 7000 (1.7 waves per SIMD) 131 -> 141, 8 heads, n = 4000 (3.9) 164 -> 127; group 3, 2
//     heads, n = 7000 (1.3) 128 -> 135; group 2, 8 heads, n = 2000 / 4000 (1.0 / 2.0) 45 -> 50 / 105 -> 92; group 1, 8
//     heads, n = 4000 / 7000 (1.0 / 1.7) 75 -> 85 / 170 -> 150.  d = 64: group 1, 8 heads, n = 4000 / 9000 (1.0 / 2.2)
//     57 -> 67 / 151 -> 144; group 4, 8 heads, n = 2000 / 4000 (2.0 / 3.9) 36 -> 41 / 96 -> 89.
//   - Of about equal length (behind a longer cache): what does not fit at once comes as a whole round more.  One 32-row
//     wave per SIMD, all workgroups resident (LDS ring: three per CU, of four waves two; d = 64 and one wave: six):
//     3000 cached tokens, d = 128: group 1, 32 heads, n = 700 (2.75 workgroups per CU) 77 -> 89, n = 1021 (4) 132 -> 100;
//     group 2, 8 heads, n = 2000 (1.0 waves per SIMD) 118 -> 102; group 4, 8 heads, n = 700 / 2000 (0.7 / 2.0) 74 -> 79 /
//     155 -> 130.  Or where this kernel would need a second round and the 32-row form would not: group 3, 32 heads,
//     n = 700 152 -> 166.
// The lines were drawn with the former main loop (which took 57, 159, 122 and 94 us where 50, 135, 102 and 79 stand now), so
// the 32-row form keeps a little too much: group 2, 8 heads, n = 2000 behind 3000 (15 %) and d = 64, group 1, n = 9000 (5 %).
// More than four query heads per KV head: this kernel at any size.  Its former main loop against the 32-row form with five to
// eight waves that it took the place of, 4000 cached tokens, n = 32: group 5 / 6 / 7 / 8 108 -> 97 / 107 -> 97 / 111 -> 97 /
// 113 -> 97; empty cache, n = 700: 36 -> 31 / 34 -> 29 / 35 -> 30 / 36 -> 30 (5 us of each for the shorter front end).
// Four waves per workgroup once every CU gets two of them, else two waves for the finer grain (8 sequences of 333 tokens:
// 29 against 31 us), unless the finer grain spills into a round of its own (group 3, 32 heads, 2500 cached tokens, n = 677:
// 544 workgroups of two waves 141 us, 256 of four 105); d = 64 is faster with four throughout (40 against 47 us with the
// former loop).
int prefill_wide_waves(int head_dim, int group, int64_t units, int max_new, int max_seq_len, int num_cus)
{
    const int64_t cus = num_cus;
    auto items_of = [&](int tokens) { return units * ((max_new + tokens - 1) / tokens); };
    const int64_t items4 = items_of(256 / group);
    const bool even = max_seq_len >= 2 * (int64_t)max_new;
    if (group <= 4) {
        const int64_t items32 = items_of(32), waves32 = items32 * group;
        const bool thin = head_dim == 64 && group == 1;
        if (!even) {
            if (waves32 <= (head_dim == 64 ? 10 : group <= 2 ? 6 : 8) * cus) return 0;
        } else if (items32 < (thin ? 6 : group <= 3 ? 3 : 2) * cus && (waves32 <= (thin ? 6 : 4) * cus || items4 > cus)) {
            return 0;
        }
    }
    if (head_dim == 64 || items4 >= 2 * cus) return 4;
    return even && (items_of(128 / group) + 2 * cus - 1) / (2 * cus) > (items4 + cus - 1) / cus ? 4 : 2;
}

hipError_t launch_prefill_attn(const AttnArgs &a, int head_dim, int num_cus, hipStream_t stream)
{
    if (a.batch == 0 || a.max_new == 0) return hipSuccess;
    const int waves = prefill_wide_waves(head_dim, a.group, (int64_t)a.batch * a.num_kv_heads, a.max_new, a.max_seq_len, num_cus);
    if (waves == 0) return launch_prefill_split(a, head_dim, num_cus, stream);
    if (head_dim == 128) return waves == 2 ? launch_prefill_wide<128, 2>(a, num_cus, stream) : launch_prefill_wide<128, 4>(a, num_cus, stream);
    if (head_dim == 64) return launch_prefill_wide<64, 4>(a, num_cus, stream);
    return hipErrorInvalidValue;
}

}  // namespace orthrus
