// Split-KV block attention for the Orthrus dual-view decode step on gfx950 (Section 3.1, Eq. 4:
// O = Softmax(Q [K_AR || K_blk]^T * scale) [V_AR || V_blk]; diffusion view bidirectional inside
// the block, AR verification view causal inside the block).
//
// Work decomposition
//   grid   = one workgroup per (split, KV head g, sequence b).  A workgroup streams its piece of the
//            cache tokens of KV head g once (the sequence's own tiles, the in-block tile included, dealt
//            out evenly to the splits: split_cut) and serves all R = G*K
//            query rows that share that KV head (G query heads x K block rows).
//            Workgroups are numbered with the sequence index fastest and the KV head slowest
//            (consecutive ids go to different XCDs; see the kernel).
//   waves  = W compute waves per workgroup, one per block of 32 query rows (W = 1 .. 8), plus
//            one loader wave.  Every compute wave reads every K/V tile, so the tile stream is shared:
//            the loader sends 32-token tiles from global memory straight into an NS-stage LDS ring
//            (global_load_lds_dwordx4: coalesced 16-byte loads, one 256-byte row per 16 lanes), NS-1
//            tiles ahead of the one being computed, with one workgroup barrier per tile.  For a
//            launch that can fill the chip the plan lands on one workgroup per CU: that keeps ~32 KB
//            in flight per CU, which already saturates HBM, and shares the bandwidth evenly between
//            the XCDs (with twice as much in flight some XCDs finish 20 % later than others); a
//            smaller launch trades the length of a workgroup's tile chain against the cost of more
//            pieces (plan_attn).
//   MFMA   = v_mfma_f32_32x32x16_bf16 for both contractions, on the transposed problem:
//            S^T[token][row] = K_tile . Q^T   (A = K from LDS, B = Q held in registers)
//            O^T[d][row]    += V^T . P^T      (A = V through the LDS transpose read, B = P)
//            In both results a lane owns one query row (lane%32), so the online-softmax row
//            statistics are per-lane scalars and need a single cross-lane exchange (lane^32).
//   tail   = the block's own K/V rows form one more 32-token tile, masked per view, processed by
//            the unit's last piece.  A wave owns its rows outright, so there is no merge inside the workgroup:
//            it writes final bf16 rows (one split) or an fp32 partial in register order that
//            attn_combine_kernel merges in a fixed split order (deterministic).
//   other forms of the same kernel: the balanced partition of a ragged batch's tiles over the
//            resident workgroups (MODE kItemsBalanced) and the AR view's causal prefill (kItemsPrefill);
//            both are described at the kernel.  Calls of at most 16 rows, and launches whose long items
//            start first, are in orthrus_attn_forms.hip.
//   caches = K/V tiles are read once per call.  When the model streams more K/V between two passes
//            over the same cache than the last-level cache holds, the tile loads carry the
//            non-temporal hint, and with fixed splits the fp32 partials leave with non-temporal stores.
#include "orthrus_attn_dev.h"

namespace orthrus {

// D head_dim, W compute waves (= 32-row blocks) per workgroup, NS LDS stages.
//
// A workgroup has W compute waves and one loader wave that issues every tile load and does nothing
// else.  A wave that issues global->LDS loads is held up while the memory pipeline takes them
// (streaming 2 MB per CU costs the issuing wave about as long as the arithmetic on it costs a compute
// wave), so when compute waves issue their own loads the two costs add up; with a dedicated loader
// wave they overlap.  The register budget is 168 (three waves per SIMD), so W + 1 <= 9 waves fit a CU;
// the balanced form at d = 128 spills five vector registers that live across segments, outside the tile loop, the others none.
//
// MODE kItemsPrefill turns the same kernel into the AR view's causal prefill attention (Section 3.1): the new
// tokens' K/V rows are already in the cache, a work item is (sequence, chunk of 32 new tokens, KV head),
// its R = 32*G rows are the chunk's tokens times the G query heads, row (token i) sees cache tokens
// 0 .. L+i (its own position included), and there is no staged block tile and no split.
//
// MODE kItemsBalanced (decode only) replaces the fixed (sequence, split, head) grid by an even partition of
// the whole launch's tile sequence: the tiles of all (head, sequence) units, cache tiles then the
// in-block tile, are laid end to end (head-major), and workgroup w of the N launched takes tiles
// [w*T/N, (w+1)*T/N).  A workgroup's range is cut into segments at unit boundaries; a segment that
// covers its whole unit writes final rows, any other writes a partial (slot 2w when it starts inside
// the unit, 2w+1 when it starts at the unit's first tile: a range holds at most one of each), which
// attn_combine_kernel finds again from the same arithmetic.  With ragged lengths every workgroup
// still gets the same number of tiles, and with N = resident workgroups nothing queues behind
// the dispatcher.  Each segment runs the pipeline from empty (fill, loop, drain).
//
// PROBE = 1 is the measurement form behind orthrus_kv_stream_probe: the loader wave streams exactly the
// tiles of the call, the compute waves only keep the barriers (no queries, no arithmetic, nothing is
// written), so the launch takes as long as this kernel's K/V stream alone.
//
// NT: the non-temporal forms of the tile loads and of the partials' stores.  A form of the kernel and not a test in it:
// every jump into code that no wave of the launch has fetched yet is a round trip to the L2 or beyond, in the loader's
// first tile and between the last tile and the write-out alike.  The balanced partition's one form (kNtAsked) has both copies
// of the loader's loop and a test: as two forms the compiler spills more of what lives across its segments (35 scalar
// registers where it is 28 at 64 rows), 15 sequences of 71..1147 tokens, 16 rows 19.5 -> 20.3 us, 4 of 300..4000, 64 rows 25.1
// -> 25.6.
// The stores' hint is for fixed splits only: there the write-back of the partials at the kernel's end is what the merge waits
// for (cycles over 12 layers of 4096 tokens at batch 4 / 8 496 -> 479 / 731 -> 711 us, 36 layers at batch 1 942 -> 940; a
// small call under a loose bound 12.1 -> 12.5).  The balanced partition writes partials all along and reads them out of the
// L2 again (64 sequences of 500..4000 tokens 133 -> 138 us with the hint).
template <int D, int W, int NS, int MODE, int NT, int PROBE = 0>
__global__ void __launch_bounds__(64 * (W + 1), 3) attn_split_kernel(ATTN_FIRST_PARAMS, const AttnArgs rest)
{
    constexpr int ROWS = 32;
#include "orthrus_attn_split.inc"
}

// Merge the per-split partials in split order and write bf16 rows.  One workgroup per (sequence,
// KV head, 32-row block, 32-wide d block), one wave per group of 4 d values: a lane reads exactly the
// float4 it would hold in the split kernel's accumulator, so every load is a contiguous 1 KB per wave
// and all splits of a chunk are in flight together.
//
// BALANCED: the pieces of a unit are found from the split kernel's partition arithmetic: unit (g, b) covers
// tiles [U0, U1) of the launch's tile sequence, its pieces belong to workgroups w_lo..w_hi, the first in its
// slot 2w+1 and the others in slot 2w; a unit held by one workgroup was finished by the split kernel.
//
// CHUNK = partials merged per round of loads: 8 keeps the registers low for the bandwidth-bound merges
// of many units with few pieces each; 16 or 32 make the latency-bound merge of few units with many
// splits a single memory round trip (a second round costs it ~1 us).
//
// WAVES = waves per workgroup: 4, or 1 where the launch would have few workgroups.  A CU pulls in some 50 KB per
// microsecond, and 64 workgroups of four waves want 100 KB each of 26 pieces (launch_combine).
template <int D, int W, int BALANCED, int CHUNK, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) attn_combine_kernel(ATTN_FIRST_PARAMS, const AttnArgs rest)
{
    const AttnArgs a = with_first(rest, first_lens, first_batch);
    static_assert(WAVES == 4 || WAVES == 1, "the four waves of a row and d block share a workgroup or have one each");
    constexpr int DBLK = D / 32;
    constexpr int MCHUNK = 32;  // m values fetched per round when there are more than CHUNK partials
    const int lane = threadIdx.x & 63, r4 = WAVES == 4 ? threadIdx.x >> 6 : blockIdx.x & 3;
    const int col = lane & 31, h = lane >> 5;
    const unsigned block = WAVES == 4 ? blockIdx.x : blockIdx.x >> 2;
    const int db = (int)(block % DBLK);
    const int wave = (int)(block / DBLK % W);  // row block
    const int unit = (int)(block / (DBLK * W));
    const int b = unit / a.num_kv_heads, g = unit % a.num_kv_heads;
    const int ridx = wave * 32 + col;
    // One row block: a padding row's lanes read the last row's data again, nothing more moves.  (More blocks are mostly rows, and
    // the minimum in front of the loads costs: 36-layer graph, 64 rows, 942 -> 954 us a cycle.)
    const int rcol = W == 1 ? min(col, a.rows - 1) : col;
    int live;           // number of partials of this unit
    size_t first_slot;  // partial index of piece 0; piece s > 0 sits at rest_slot + s * slot_step
    size_t rest_slot, slot_step;
    if constexpr (BALANCED) {
        int before = 0, per_head = 0, mine = 0;  // tiles of the sequences before b, of all, of b
        for (int x0 = 0; x0 < a.batch; x0 += 64) {
            const int x = x0 + lane;
            int n = 0;
            if (x < a.batch) {
                int L = a.seq_lens[x];
                L = L < 0 ? 0 : (L > a.max_seq_len ? a.max_seq_len : L);
                n = ((L + 31) >> 5) + 1;
            }
            int nb = x < b ? n : 0, nm = x == b ? n : 0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                n += __shfl_xor(n, off);
                nb += __shfl_xor(nb, off);
                nm += __shfl_xor(nm, off);
            }
            per_head += n;
            before += nb;
            mine += nm;
        }
        const int64_t total = (int64_t)per_head * a.num_kv_heads;
        const int64_t nwg = total < (int64_t)a.bal_wgs ? total : (int64_t)a.bal_wgs;
        const int64_t U0 = (int64_t)g * per_head + before, U1 = U0 + mine;
        // workgroup w starts at tile floor(w * total / nwg): w_lo is the last one that starts at or
        // before U0, w_hi the last one that starts before U1
        const int64_t w_lo = ((U0 + 1) * nwg + total - 1) / total - 1;
        const int64_t w_hi = (U1 * nwg + total - 1) / total - 1;
        if (w_lo == w_hi) return;  // one workgroup held the whole unit and wrote its rows
        live = (int)(w_hi - w_lo + 1);
        first_slot = (size_t)w_lo * 2 + 1;
        rest_slot = (size_t)w_lo * 2;
        slot_step = 2;
    } else {
        live = a.num_splits;  // the slots, until the length is there
        first_slot = rest_slot = (size_t)unit * a.num_splits;
        slot_step = 1;
    }
    // partial `s` of this unit: (m, l) of the lane's row and the lane's float4 of the accumulator
    auto ml_at = [&](int s) __attribute__((always_inline)) {
        const size_t slot = (s == 0 ? first_slot : rest_slot + (size_t)s * slot_step) * W + wave;
        return (const float2 *)a.part_ml + slot * 32 + rcol;
    };
    auto po_at = [&](int s) __attribute__((always_inline)) {
        const size_t slot = (s == 0 ? first_slot : rest_slot + (size_t)s * slot_step) * W + wave;
        return (const float4 *)a.part_o + slot * (DBLK * 4 * 64) + (size_t)(db * 4 + r4) * 64 + (W == 1 ? h * 32 + rcol : lane);
    };

    // The loads of the first CHUNK partials go out before anything waits; the reference maximum needs
    // every partial's m, so the remaining m values follow MCHUNK at a time, then the rest of the data.
    // A merge of up to CHUNK partials is one memory round trip, not one per pass.
    //
    // Few units (one wave per workgroup): what counts is the chain.  With fixed splits the first loads do not wait for the
    // sequence's length, which says how many of the num_splits slots hold a piece; what the others bring is dropped.  They go
    // out in pairs, a jump to a pair.  The balanced partition cuts few units into many pieces: whole chunks without a jump,
    // the last one repeats its last piece and drops the copies.
    // Many units (four waves): what counts is the loads, so those of live pieces only, a jump to a load.
    // Per call, this form for every launch -> all CHUNK loads at once for every launch -> as it is: 16 sequences of 50..300
    // tokens under a bound of 8000 (2 splits) 11.7 -> 13.5 -> 12.4 us; 2 of 300 under 32768, 128 rows (15) 10.9 -> 11.3 ->
    // 10.8; one of 2000, 128 rows (9) 12.2 -> 12.5 -> 12.1; balanced, 64 of 500..4000 133 -> 143 -> 138 (133 with the
    // partials' plain stores); one wave: 36-layer graph, 64 rows, 4112 tokens (13), a cycle 965 -> 941 -> 940; one of 4096, 224
    // rows (22) 15.3 -> 15.6 -> 15.4; balanced, 3 of 100..4000 (d = 64, some 40 pieces) 26 -> 23.4 -> 23.3, in pairs 25.
    constexpr bool EARLY = WAVES == 1 && !BALANCED;
    constexpr int RUN = WAVES == 4 ? 1 : BALANCED ? CHUNK : 2;
    static_assert(CHUNK % RUN == 0, "");
    float4 v[CHUNK];
    float2 e[CHUNK];
    auto load_chunk = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u0 = 0; u0 < CHUNK; u0 += RUN) {
            if (s0 + u0 < live) {
#pragma unroll
                for (int u = u0; u < u0 + RUN; ++u) {
                    const int s = RUN == 1 ? s0 + u : min(s0 + u, live - 1);
                    v[u] = *po_at(s);
                    e[u] = *ml_at(s);
                }
            } else {
#pragma unroll
                for (int u = u0; u < u0 + RUN; ++u) {
                    v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                    e[u] = make_float2(kNegBig, 0.f);
                }
            }
        }
    };
    auto drop_past_end = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CHUNK; ++u) {
            if (s0 + u >= live) {
                v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                e[u] = make_float2(kNegBig, 0.f);
            }
        }
    };
    if constexpr (EARLY) {
        load_chunk(0);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!BALANCED) {
        int L = ((const const_i32 *)a.seq_lens)[b];
        L = L < 0 ? 0 : (L > a.max_seq_len ? a.max_seq_len : L);
        live = split_cut(L, a.num_splits, 0).live;  // the split kernel's pieces of this sequence
    }
    if constexpr (!EARLY) load_chunk(0);
    if constexpr (RUN > 1) drop_past_end(0);
    float M = kNegBig;
#pragma unroll
    for (int u = 0; u < CHUNK; ++u) M = fmaxf(M, e[u].x);
    for (int s0 = CHUNK; s0 < live; s0 += MCHUNK) {
        float mv[MCHUNK];
#pragma unroll
        for (int u = 0; u < MCHUNK; ++u) mv[u] = (s0 + u < live) ? ml_at(s0 + u)->x : kNegBig;
#pragma unroll
        for (int u = 0; u < MCHUNK; ++u) M = fmaxf(M, mv[u]);
    }
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float lsum = 0.f;
    for (int s0 = 0; s0 < live; s0 += CHUNK) {
        if (s0 > 0) {
            load_chunk(s0);
            if constexpr (RUN > 1) drop_past_end(s0);
        }
#pragma unroll
        for (int u = 0; u < CHUNK; ++u) {  // fixed split order: the result does not depend on timing
            const float sc = __builtin_amdgcn_exp2f(e[u].x - M);
            lsum += sc * e[u].y;
            acc.x += sc * v[u].x; acc.y += sc * v[u].y; acc.z += sc * v[u].z; acc.w += sc * v[u].w;
        }
    }
    if (ridx >= a.rows) return;
    const int G = a.group, K = a.block_k;
    const int i = ridx / G, hl = ridx - i * G;
    const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
    uint16_t *op = a.out + (((int64_t)b * K + i) * a.num_q_heads + (int64_t)g * G + hl) * D;
    uint2 pk;
    pk.x = pack_bf16(acc.x * inv, acc.y * inv);
    pk.y = pack_bf16(acc.z * inv, acc.w * inv);
    *(uint2 *)(op + 32 * db + 8 * r4 + 4 * h) = pk;
    if (a.lse && db == 0 && r4 == 0 && h == 0)
        a.lse[((int64_t)b * a.num_q_heads + (int64_t)g * G + hl) * K + i] =
            (M + __builtin_amdgcn_logf(lsum)) * 0.6931471805599453f;
}

// ---------------------------------------------------------------------------------------------
// host side

static size_t lds_need(int head_dim)
{
    return (size_t)kStages * (head_dim == 128 ? AttnGeom<128>::STAGE_B : AttnGeom<64>::STAGE_B);
}

// Workgroups of W compute waves that are resident on a CU: LDS ring size, and 12 waves (3 per SIMD: the kernel stays
// below 168 registers) of W compute waves + the loader wave each
static int resident_per_cu(int head_dim, int W)
{
    const int by_lds = (int)(160 * 1024 / lds_need(head_dim)), by_waves = 12 / (W + 1);
    return by_lds < by_waves ? by_lds : by_waves > 0 ? by_waves : 1;
}

// One wave per workgroup while four would leave most CUs without any (256 CUs, 36-layer graph, 4096 tokens, per call: 64
// workgroups of 64 rows, 15 / 26 pieces 12.8 -> 12.6 / 13.8 -> 13.1 us; from 128 on the larger number is what counts: 128 rows,
// 13 / 15 pieces 16.3 -> 16.5 / 16.0 -> 16.3; 256 of 64 rows, 8 pieces 19.7 -> 19.9).
int merge_waves(int64_t wgs, int num_cus) { return 2 * wgs < num_cus ? 1 : 4; }

bool decode_by_size(int batch, int64_t items, int per_cu, int num_cus) { return batch > 1 && items > (int64_t)per_cu * num_cus; }

int decode_direction_on_host(const int *lens, int batch, bool small_counts)
{
    int sample[kOrderSamples];
    for (int k = 0; k < kOrderSamples; ++k) sample[k] = lens[order_sample(k, batch)];
    return direction_of(sample, batch, small_counts);
}

hipError_t plan_attn(int head_dim, int group, int block_k, int batch, int num_kv_heads, int max_seq_len,
                     int requested_splits, int num_cus, int num_layers, double pool_tokens, AttnPlan *plan)
{
    const int R = group * block_k;
    plan->rows = R;
    const int blocks = R > 32 ? (R + 31) / 32 : 1;
    const int64_t units = (int64_t)batch * num_kv_heads;
    plan->wide = requested_splits >= 0 && requested_splits <= 1 && attn_wide_pays(head_dim, R, max_seq_len, units, num_cus);
    const int W = plan->wide ? (R > 128 ? 4 : 2) : blocks;
    plan->waves = W;
    plan->rows_padded = blocks * 32;
    plan->lds_bytes = plan->wide ? attn_wide_lds(W, head_dim) : lds_need(head_dim);
    const int per_cu = plan->wide ? attn_wide_per_cu(W) : resident_per_cu(head_dim, W);  // resident workgroups
    plan->merge_waves = merge_waves(units * W * (head_dim / 32), num_cus);
    plan->bal_wgs = 0;
    plan->by_size = 0;
    // K/V bytes the model streams at most between two passes over the same layer's cache (the other
    // layers' caches come in between), against the 256 MB last-level cache (see the kernel's loads).  Sequences
    // may share pages: a layer holds no more tokens than its pool (the training mask's 1024 blocks read 32 MB
    // between them: 685 us with non-temporal loads, 622 without; 64 caches of their own 89 against 99).
    const double tokens = (double)batch * max_seq_len < pool_tokens ? (double)batch * max_seq_len : pool_tokens;
    const double stream_bytes = (double)(num_layers > 1 ? num_layers : 1) * tokens * num_kv_heads * 4.0 * head_dim;
    plan->kv_nt = stream_bytes > 1.25 * 256.0 * 1024 * 1024 ? 1 : 0;
    if (requested_splits < 0) {
        // balanced partition: as many workgroups as are resident at once, two partial slots each
        plan->bal_wgs = num_cus * per_cu;
        plan->chunk_tokens = 32;
        plan->num_splits = 1;
        plan->part_o_bytes = (size_t)plan->bal_wgs * 2 * plan->rows_padded * head_dim * sizeof(float);
        plan->part_ml_bytes = (size_t)plan->bal_wgs * 2 * plan->rows_padded * 2 * sizeof(float);
        return hipSuccess;
    }
    int splits;
    if (plan->wide) {
        splits = 1;  // its units alone fill the chip
    } else if (requested_splits > 0) {
        splits = requested_splits;
    } else {
        // Pick the split count with a small cost model (times in microseconds, constants measured on
        // this chip), using max_seq_len for every sequence.  Workgroups run in rounds of `slots`.  A
        // workgroup needs at least kTile per 32-token tile whatever the stream could deliver (the
        // loader wave's issue rate and the dependent chain of one tile's products and softmax are
        // both about that long: what binds when few CUs are busy, e.g. batch 1), and the tiles of all
        // workgroups of a round together stream no faster than kRate.  Every workgroup costs kWg to
        // dispatch; every piece beyond a unit's first is an fp32 partial (rows x d x 4 bytes) written
        // once and read once, and brings the merge launch with it.  The constants are part of the interface: programs
        // keep the workspace that the split count asks for, and each piece rounds its weights against its own
        // reference, so that another count gives other bits.
        const double kRate = 7.0e6;      // K/V bytes per microsecond (measured ceiling of the paged stream)
        const double kPartRate = 6.0e6;  // bytes per microsecond for the partials
        const double kTile = W <= 4 ? 0.56 : 1.3;  // more than four 32-row blocks: two per SIMD
        const double kRound = 5.0, kCombine = 4.0, kSplit = 0.12, kWg = 0.008;
        const int64_t slots = (int64_t)num_cus * per_cu;
        const double tile_bytes = 32.0 * 2.0 * head_dim * 2.0;  // K + V bytes of one tile of one KV head
        const double part_bytes = 2.0 * plan->rows_padded * head_dim * 4.0;  // written once, read once
        const int max_s = max_seq_len >= 256 ? (max_seq_len / 128 < 64 ? max_seq_len / 128 : 64) : 1;
        const int tiles = (max_seq_len + 31) / 32;
        double cost[65];
        double best = 1e300;
        for (int s = 1; s <= max_s; ++s) {
            const int64_t wgs = units * s;
            const double tiles_per_wg = (double)((tiles + s - 1) / s);
            double t = s > 1 ? kCombine + kSplit * s : 0.0;  // the merge reads one more partial per output and split
            for (int64_t left = wgs; left > 0; left -= slots) {
                const int64_t now = left < slots ? left : slots;
                const double per_tile = tile_bytes * now / kRate;  // all workgroups of the round share the stream
                t += kRound + tiles_per_wg * (per_tile > kTile ? per_tile : kTile) +
                     now * (kWg + (s > 1 ? part_bytes / kPartRate : 0.0));
            }
            cost[s] = t;
            if (t < best) best = t;
        }
        splits = 1;
        while (cost[splits] > best * 1.01) ++splits;  // the fewest splits within 1 % of the best estimate
    }
    int chunk = (max_seq_len + splits - 1) / splits;
    chunk = ((chunk + 31) / 32) * 32;
    if (chunk < 32) chunk = 32;
    splits = max_seq_len > 0 ? (max_seq_len + chunk - 1) / chunk : 1;
    if (splits < 1) splits = 1;
    plan->chunk_tokens = chunk;
    plan->num_splits = splits;
    plan->by_size = decode_by_size(batch, units * splits, per_cu, num_cus) ? 1 : 0;
    if (splits > 1) {
        plan->part_o_bytes = (size_t)units * splits * plan->rows_padded * head_dim * sizeof(float);
        plan->part_ml_bytes = (size_t)units * splits * plan->rows_padded * 2 * sizeof(float);
    } else {
        plan->part_o_bytes = plan->part_ml_bytes = 0;
    }
    return hipSuccess;
}

template <int D, int W, int BALANCED>
static hipError_t launch_split(const AttnArgs &a, const AttnPlan &plan, dim3 grid, hipStream_t stream, AttnLaunchEvents *ev)
{
    if (a.rows <= 16) return launch_attn_thin(a, plan, D, grid, stream, ev);
    if (plan.by_size) return launch_attn_by_size(a, plan, D, grid, stream, ev);
    auto kern = [&] {
        if constexpr (BALANCED) return attn_split_kernel<D, W, kStages, kItemsBalanced, kNtAsked>;
        else return plan.kv_nt ? attn_split_kernel<D, W, kStages, kItemsSplit, 1> : attn_split_kernel<D, W, kStages, kItemsSplit, 0>;
    }();
    return launch_timed(kern, grid, dim3(64 * (W + 1)), plan.lds_bytes, a, stream, ev, 0);
}

template <int D, int W, int BALANCED, int WAVES>
static auto combine_kernel(int num_splits)
{
    if constexpr (!BALANCED) {
        if (num_splits > 16) return attn_combine_kernel<D, W, 0, 32, WAVES>;
        if (num_splits > 8) return attn_combine_kernel<D, W, 0, 16, WAVES>;
    }
    return attn_combine_kernel<D, W, BALANCED, 8, WAVES>;
}

template <int D, int W, int BALANCED>
static hipError_t launch_combine(const AttnArgs &a, const AttnPlan &plan, hipStream_t stream, AttnLaunchEvents *ev)
{
    const unsigned wgs = (unsigned)(a.batch * a.num_kv_heads) * W * (D / 32);
    if (plan.merge_waves == 1) return launch_timed(combine_kernel<D, W, BALANCED, 1>(a.num_splits), dim3(wgs * 4), dim3(64), 0, a, stream, ev, 1);
    return launch_timed(combine_kernel<D, W, BALANCED, 4>(a.num_splits), dim3(wgs), dim3(256), 0, a, stream, ev, 1);
}

// One attention call: the split kernel, then the merge when units were cut into pieces.
template <int D, int BALANCED>
static hipError_t launch_attn_d(const AttnArgs &a, const AttnPlan &plan, hipStream_t stream, AttnLaunchEvents *ev)
{
    dim3 grid(BALANCED ? (unsigned)plan.bal_wgs
                       : (unsigned)plan.num_splits * (unsigned)a.num_kv_heads * (unsigned)a.batch);
    hipError_t e = hipErrorInvalidValue;
    if (plan.wide) {
        e = launch_attn_wide(a, plan, D, grid, stream, ev);
    } else {
        switch (plan.waves) {
        case 1: e = launch_split<D, 1, BALANCED>(a, plan, grid, stream, ev); break;
        case 2: e = launch_split<D, 2, BALANCED>(a, plan, grid, stream, ev); break;
        case 3: e = launch_split<D, 3, BALANCED>(a, plan, grid, stream, ev); break;
        case 4: e = launch_split<D, 4, BALANCED>(a, plan, grid, stream, ev); break;
        case 5: e = launch_split<D, 5, BALANCED>(a, plan, grid, stream, ev); break;
        case 6: e = launch_split<D, 6, BALANCED>(a, plan, grid, stream, ev); break;
        case 7: e = launch_split<D, 7, BALANCED>(a, plan, grid, stream, ev); break;
        case 8: e = launch_split<D, 8, BALANCED>(a, plan, grid, stream, ev); break;
        }
    }
    if (e != hipSuccess) return e;
    if (BALANCED || plan.num_splits > 1) {
        switch (plan.waves) {
        case 1: e = launch_combine<D, 1, BALANCED>(a, plan, stream, ev); break;
        case 2: e = launch_combine<D, 2, BALANCED>(a, plan, stream, ev); break;
        case 3: e = launch_combine<D, 3, BALANCED>(a, plan, stream, ev); break;
        case 4: e = launch_combine<D, 4, BALANCED>(a, plan, stream, ev); break;
        case 5: e = launch_combine<D, 5, BALANCED>(a, plan, stream, ev); break;
        case 6: e = launch_combine<D, 6, BALANCED>(a, plan, stream, ev); break;
        case 7: e = launch_combine<D, 7, BALANCED>(a, plan, stream, ev); break;
        case 8: e = launch_combine<D, 8, BALANCED>(a, plan, stream, ev); break;
        }
    }
    return e;
}

// The stream probe: the same grid, partition and loader as the attention call planned by `plan`, with one
// idle compute wave per workgroup and the items in the plain order.
template <int D>
static hipError_t launch_probe_d(const AttnArgs &a, const AttnPlan &plan, hipStream_t stream, hipEvent_t start,
                                 hipEvent_t stop)
{
    const bool bal = plan.bal_wgs > 0;
    auto kern = plan.kv_nt ? (bal ? attn_split_kernel<D, 1, kStages, kItemsBalanced, 1, 1> : attn_split_kernel<D, 1, kStages, kItemsSplit, 1, 1>)
                           : (bal ? attn_split_kernel<D, 1, kStages, kItemsBalanced, 0, 1> : attn_split_kernel<D, 1, kStages, kItemsSplit, 0, 1>);
    dim3 grid(bal ? (unsigned)plan.bal_wgs : (unsigned)plan.num_splits * (unsigned)a.num_kv_heads * (unsigned)a.batch);
    const size_t lds = lds_need(D);
    if (start && stop) hipExtLaunchKernelGGL(kern, grid, dim3(128), lds, stream, start, stop, 0, ATTN_FIRST_VALUES(a), a);
    else hipLaunchKernelGGL(kern, grid, dim3(128), lds, stream, ATTN_FIRST_VALUES(a), a);
    return hipGetLastError();
}

hipError_t launch_kv_stream_probe(const AttnArgs &a, const AttnPlan &plan, int head_dim, hipStream_t stream,
                                  hipEvent_t start, hipEvent_t stop)
{
    if (a.batch == 0) return hipSuccess;
    if (head_dim == 128) return launch_probe_d<128>(a, plan, stream, start, stop);
    if (head_dim == 64) return launch_probe_d<64>(a, plan, stream, start, stop);
    return hipErrorInvalidValue;
}

// The prefill form with a compute wave per query head of the group (see launch_prefill_attn).  Ordinary loads: every chunk
// of a sequence reads the same cache rows again.
template <int D>
static hipError_t launch_prefill_split_d(AttnArgs a, int num_cus, hipStream_t stream)
{
    a.chunk_tokens = 32;
    a.rows = 32 * a.group;
    a.num_splits = (a.max_new + 31) / 32;
    dim3 grid((unsigned)a.num_splits * (unsigned)a.num_kv_heads * (unsigned)a.batch);
    a.ranked = prefill_ranked(a.batch, grid.x, resident_per_cu(D, a.group), num_cus);
    auto kern = a.group == 1   ? attn_split_kernel<D, 1, kStages, kItemsPrefill, 0>
                : a.group == 2 ? attn_split_kernel<D, 2, kStages, kItemsPrefill, 0>
                : a.group == 3 ? attn_split_kernel<D, 3, kStages, kItemsPrefill, 0>
                               : attn_split_kernel<D, 4, kStages, kItemsPrefill, 0>;
    hipLaunchKernelGGL(kern, grid, dim3(64 * (a.group + 1)), lds_need(D), stream, ATTN_FIRST_VALUES(a), a);
    return hipGetLastError();
}

hipError_t launch_prefill_split(const AttnArgs &a, int head_dim, int num_cus, hipStream_t stream)
{
    if (a.group > 4) return hipErrorInvalidValue;
    if (head_dim == 128) return launch_prefill_split_d<128>(a, num_cus, stream);
    if (head_dim == 64) return launch_prefill_split_d<64>(a, num_cus, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_attn(const AttnArgs &a, const AttnPlan &plan, int head_dim, hipStream_t stream,
                       AttnLaunchEvents *events)
{
    if (a.batch == 0) return hipSuccess;
    const bool bal = plan.bal_wgs > 0;
    if (head_dim == 128)
        return bal ? launch_attn_d<128, 1>(a, plan, stream, events) : launch_attn_d<128, 0>(a, plan, stream, events);
    if (head_dim == 64)
        return bal ? launch_attn_d<64, 1>(a, plan, stream, events) : launch_attn_d<64, 0>(a, plan, stream, events);
    return hipErrorInvalidValue;
}

}  // namespace orthrus
