// Device code shared by the attention kernels: operand types, the LDS tile layout, the direct-to-LDS loads and the
// walk over a launch's work items.
#pragma once
#include "orthrus_internal.h"

#include <hip/hip_ext.h>

#include <type_traits>

#pragma clang diagnostic ignored "-Winline-asm"  // the direct-to-LDS loads below name M0 as clobbered

namespace orthrus {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(4))) int32_t const_i32;

union Frag {
    uint4 u;
    bf16x8 v;
    s16x4 h[2];
    u32x4 n;
};

// LDS tile layout.  A wave-wide 16-byte direct load fills 1024 contiguous LDS bytes = one "group" of
// RPI consecutive K/V rows; groups are GS = 1040 bytes apart (the 16 bytes of padding rotate the
// banks from group to group).  Inside a group, row r keeps its 16-byte chunk c at slot c ^ xm(r),
// xm(r) = (r << 2) mod chunks-per-row, i.e. each row of a group starts in a different 64-byte bank
// window.  Both MFMA operand read patterns then spread over the banks: the K read (lanes = 32
// consecutive rows, same chunk) and the V transpose read (16 lanes = 4 rows x 32 bytes).  The
// permutation is applied on the global side (a lane fetches the chunk that belongs in its slot).
constexpr int kGroupStride = 1040;
constexpr float kLazy = 8.0f;  // log2 of the largest exponential the lazy softmax reference allows
template <int CH>
__device__ __forceinline__ int xm(int r)
{
    return (r << 2) & (CH - 1);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // v_cvt_pk_bf16_f32, RNE
}

// A finished output row, d values 8*r4 + 4*h + 0..3 of each 32-wide block in a lane (h = lane / 32): the two lanes of a row
// trade quarters, so that each stores 16 bytes in a row (h = 0 the even eights, h = 1 the odd ones) instead of 8 twice: half
// the stores, in pieces of 32 bytes.  Both lanes of a row take part or neither does.  Training mask (268 MB of rows)
// 614 -> 600 us, over 600 tokens 295 -> 282; 512 units of 180 tokens at 128 rows 23.4 -> 21.6; 8192 new tokens 458 -> 454.
template <int DBLK, class Acc>
__device__ __forceinline__ void store_row(uint16_t *op, const Acc &o, float inv, int h)
{
#pragma unroll
    for (int db = 0; db < DBLK; ++db)
#pragma unroll
        for (int r = 0; r < 16; r += 8) {
            const uint32_t e0 = pack_bf16(o[db][r] * inv, o[db][r + 1] * inv), e1 = pack_bf16(o[db][r + 2] * inv, o[db][r + 3] * inv);
            const uint32_t o0 = pack_bf16(o[db][r + 4] * inv, o[db][r + 5] * inv), o1 = pack_bf16(o[db][r + 6] * inv, o[db][r + 7] * inv);
            const auto x = __builtin_amdgcn_permlane32_swap(e0, o0, false, false), y = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
            *(uint4 *)(op + 32 * db + 2 * r + 8 * h) = make_uint4(x[0], y[0], x[1], y[1]);
        }
}

// Combine a value with the one held by lane ^ 32 (the other half-wave) without going through LDS:
// v_permlane32_swap exchanges the upper half of one register with the lower half of another.
__device__ __forceinline__ float max_with_other_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_other_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same with lane ^ 16.
__device__ __forceinline__ float max_with_other_row(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_with_other_row(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Online softmax of one lane's 16 scores (half of a row; lane ^ 32 holds the rest) against a lazily updated
// reference m in the log2 domain.  The weights are taken against the old reference first.  Only when their sum says
// that one of them may have outgrown it by more than 2^kLazy (rarely, after a row's first tile) is the maximum taken,
// and the reference moves to it by the same rule that a maximum in every tile would apply: no maximum on the common
// path (about 15 of the 75 vector instructions a tile would cost) and the same bits.  A weight above 2^kLazy puts the
// sum above kLazySum (a little below 2^kLazy, for the exponential's rounding); a sum that is NaN compares false.  (A
// row whose later tiles all score 4 to 8 octaves above its first one has its maximum taken in every tile.)
constexpr float kLazySum = 255.0f;
static_assert(kLazy == 8.0f, "kLazySum follows it");
__device__ __forceinline__ void row_weights(const f32x16 &s, float c, float m, float (&e)[16], float &sum)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -m));
    sum = e[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) sum += e[r];
}
__device__ __forceinline__ bool may_outgrow(float sum) { return __any(!(sum <= kLazySum)); }
// Moves m to the running maximum of the row if any of the wave's rows has outgrown its reference, and takes the weights
// again; alpha is the factor for the sums so far.  False when nothing moved.
__device__ __forceinline__ bool move_reference(const f32x16 &s, float c, float &m, float (&e)[16], float &sum, float &alpha)
{
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    const float m_cand = fmaxf(m, max_with_other_half(mx) * c);
    if (!__any(m_cand - m > kLazy)) return false;
    alpha = __builtin_amdgcn_exp2f(m - m_cand);
    m = m_cand;
    row_weights(s, c, m, e, sum);
    return true;
}

// Plain workgroup barrier.  Tile loads are tracked by hand (vmcnt), LDS traffic of the compiler's own
// instructions is complete once their results were consumed; the empty asm statements keep the
// compiler from moving memory operations across the barrier.
__device__ __forceinline__ void wg_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The tiles of one (sequence, KV head) unit, cache tiles of 32 tokens followed by the in-block tile, dealt
// out to `splits` pieces as evenly as whole tiles allow: the first `rem` pieces get one tile more, pieces
// past the tile count get nothing, and the in-block tile (the unit's last) lands in the last piece that
// has any.  A launch ends with its longest piece and the others cannot make up for it (a lone CU streams
// no faster when its neighbours are done), so one tile of imbalance costs a whole tile's time.
struct SplitCut {
    int first;  // first tile of the piece (tile index in the unit)
    int count;  // tiles in it, the in-block tile included if it is the unit's last piece
    int live;   // pieces of this unit that have any tile
};
__host__ __device__ __forceinline__ SplitCut split_cut(int L, int splits, int split)
{
    const int total = ((L + 31) >> 5) + 1;  // cache tiles + the in-block tile
    const int per = total / splits, rem = total - per * splits;
    SplitCut c;
    c.first = split * per + (split < rem ? split : rem);
    c.count = per + (split < rem ? 1 : 0);
    c.live = total < splits ? total : splits;
    return c;
}

template <int D>
struct AttnGeom {
    static constexpr int CH = D / 8;          // 16-byte chunks per K/V row
    static constexpr int ROWB = D * 2;        // bytes per K/V row
    static constexpr int RPI = 64 / CH;       // rows per group = rows fetched by one wave-wide 16-byte load
    static constexpr int NI = 32 / RPI;       // groups (= such loads) per 32-token K (or V) tile
    static constexpr int GS = kGroupStride;   // LDS bytes between groups
    static constexpr int TILE_B = NI * GS;    // one 32-token K (or V) tile in LDS
    static constexpr int STAGE_B = 2 * TILE_B;
    static constexpr int KSTEPS = D / 16;     // MFMA steps along d for S
    static constexpr int DBLK = D / 32;       // 32-wide output blocks along d
};


// What the first dependent load (the length, then page ids, then tiles) hangs on stands once more in front of the struct, as
// plain values: the dispatch puts those into scalar registers before a wave starts (the build's kernarg-preload option), so
// that load goes out next to the struct's and not behind it.  No more than that: each argument costs the host some 20 ns a
// launch (eight of them made a small call of two launches 8.7 -> 9.1 us).
#define ATTN_FIRST_PARAMS const int32_t *first_lens, int first_batch
#define ATTN_FIRST_VALUES(a) (a).seq_lens, (a).batch
__device__ __forceinline__ AttnArgs with_first(AttnArgs a, ATTN_FIRST_PARAMS)
{
    a.seq_lens = first_lens;
    a.batch = first_batch;
    return a;
}

// A pointer that is uniform by construction; readfirstlane keeps the compiler from carrying it in vector registers.
__device__ __forceinline__ const void *uniform_ptr(const void *p)
{
    return (const void *)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)p) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)p >> 32)) << 32);
}

// Direct global->LDS load of 64 x 16 bytes: lane's bytes land at lds_addr + lane*16.  Issued through inline assembly so
// that whole tiles can stay in flight while older ones are computed; completion is awaited explicitly with s_waitcnt
// vmcnt (loads return in order).  M0 carries the LDS destination and is declared clobbered, so the compiler never
// carries a value of its own in M0 across one of these statements (M0 is a reserved register, which clang remarks on
// for any clobber list that names it; the remark is switched off for these files).
//
// NT selects the non-temporal form of the loads: when one call streams more K/V than the last-level cache holds,
// nothing of it is there for the next call anyway, and loads that do not allocate on their way stream ~7 % faster
// (measured); a working set that fits keeps the plain form, so that the second view's pass over the same cache still
// finds it.
template <class NT>
__device__ __forceinline__ void dma16(NT, const uint16_t *gp, uint32_t lds_addr)
{
    if constexpr (NT::value)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(gp), "s"(lds_addr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gp), "s"(lds_addr) : "memory", "m0");
}

// The same with a wave-uniform base and a 32-bit byte offset per lane.  A vector-memory instruction may read a scalar
// register five wait states after a vector instruction has written it (a lane read, from which a base comes whenever the
// compiler holds it in vector registers).  The compiler keeps that distance for its own instructions, not into an assembly
// statement, so the statement brings it along: the write of M0 is one, s_nop 3 the other four.
template <class NT>
__device__ __forceinline__ void dma16s(NT, const uint16_t *base, uint32_t voff, uint32_t lds_addr)
{
    base = (const uint16_t *)uniform_ptr(base);
    if constexpr (NT::value)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}

// The loads of whole 16-token halves of a K or V tile (a half lies inside one page): a wave-uniform base (page, head,
// token: scalar arithmetic on 32-bit byte strides) plus a loop-invariant byte offset per lane.  A half is GPH wave-wide
// loads into groups GS bytes apart.  The instruction offset e*GS moves the LDS side and the memory side of load e
// alike, so one M0 value serves the half and the lane offsets take e*GS back (the base is lowered by kBias so that
// they stay positive).  One load costs the issuing wave two instructions instead of the ~11 of 64-bit arithmetic per load.
// The wait inside the statements is that of dma16s.
template <int D>
struct HalfLoads {
    using Gm = AttnGeom<D>;
    static constexpr int GPH = Gm::NI / 2;                 // loads per half
    static constexpr uint32_t kBias = (GPH - 1) * Gm::GS;
    uint32_t voff[GPH];
    uint32_t page_bytes, tok_bytes, page_mask, num_pages;
    uint32_t worst = 0;  // largest page id seen (as unsigned); an id past num_pages was read as page 0
    bool usable;         // the strides fit the 32-bit arithmetic

    __device__ __forceinline__ HalfLoads(const AttnArgs &a, int lane)
    {
        usable = a.stride_page < (1ll << 31) && a.stride_tok < (1ll << 30) >> a.page_shift;
        page_bytes = (uint32_t)a.stride_page * 2u;
        tok_bytes = (uint32_t)a.stride_tok * 2u;
        page_mask = (1u << a.page_shift) - 1u;
        num_pages = (uint32_t)min(a.num_pages, (int64_t)0x7fffffff);
        const int tok = lane / Gm::CH, ch = lane % Gm::CH;
#pragma unroll
        for (int e = 0; e < GPH; ++e)
            voff[e] = kBias - e * Gm::GS + (uint32_t)(tok + e * Gm::RPI) * tok_bytes + (uint32_t)((ch ^ xm<Gm::CH>(tok)) << 4);
    }
    // byte offset of token position `tok` (a multiple of 16) behind page id `id`
    __device__ __forceinline__ uint64_t offset(int id, uint32_t tok)
    {
        worst = max(worst, (uint32_t)id);
        const uint32_t pg = (uint32_t)id < num_pages ? (uint32_t)id : 0u;
        return (uint64_t)pg * page_bytes + (tok & page_mask) * tok_bytes;
    }
    static __device__ __forceinline__ const char *lowered(const uint16_t *pool) { return (const char *)pool - kBias; }
    // SETTLED: the caller keeps the distance from a lane read
    template <bool SETTLED = false, class NT>
    __device__ __forceinline__ void issue(NT, const char *base, uint32_t lds_addr) const
    {
        base = (const char *)uniform_ptr(base);
        constexpr int WAIT = SETTLED ? 0 : 3;
        static_assert(Gm::GS == 1040 && (GPH == 4 || GPH == 2), "the instruction offsets below");
        if constexpr (GPH == 4 && NT::value)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop %6\n\t"
                         "global_load_lds_dwordx4 %2, %1 nt\n\tglobal_load_lds_dwordx4 %3, %1 offset:1040 nt\n\t"
                         "global_load_lds_dwordx4 %4, %1 offset:2080 nt\n\tglobal_load_lds_dwordx4 %5, %1 offset:3120 nt"
                         : : "s"(lds_addr), "s"(base), "v"(voff[0]), "v"(voff[1]), "v"(voff[GPH - 2]), "v"(voff[GPH - 1]), "n"(WAIT) : "memory", "m0");
        else if constexpr (GPH == 4)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop %6\n\t"
                         "global_load_lds_dwordx4 %2, %1\n\tglobal_load_lds_dwordx4 %3, %1 offset:1040\n\t"
                         "global_load_lds_dwordx4 %4, %1 offset:2080\n\tglobal_load_lds_dwordx4 %5, %1 offset:3120"
                         : : "s"(lds_addr), "s"(base), "v"(voff[0]), "v"(voff[1]), "v"(voff[GPH - 2]), "v"(voff[GPH - 1]), "n"(WAIT) : "memory", "m0");
        else if constexpr (NT::value)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop %4\n\t"
                         "global_load_lds_dwordx4 %2, %1 nt\n\tglobal_load_lds_dwordx4 %3, %1 offset:1040 nt"
                         : : "s"(lds_addr), "s"(base), "v"(voff[0]), "v"(voff[1]), "n"(WAIT) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop %4\n\t"
                         "global_load_lds_dwordx4 %2, %1\n\tglobal_load_lds_dwordx4 %3, %1 offset:1040"
                         : : "s"(lds_addr), "s"(base), "v"(voff[0]), "v"(voff[1]), "n"(WAIT) : "memory", "m0");
    }
};

// The 2*NI loads of a whole K/V tile whose rows are addressed lane by lane: row_off(u) is the byte offset of the row
// that the lane fetches for group u, behind a uniform base per operand and half (a row's K and V share the offset).
template <int D, class NT, class RowOff>
__device__ __forceinline__ void issue_rows(NT nt, const uint16_t *const (&k)[2], const uint16_t *const (&v)[2], uint32_t lds_addr,
                                           RowOff row_off)
{
    using Gm = AttnGeom<D>;
#pragma unroll
    for (int u = 0; u < Gm::NI; ++u) {
        const int hf = u * Gm::RPI / 16;
        const uint32_t off = row_off(u);
        dma16s(nt, k[hf], off, lds_addr + u * Gm::GS);
        dma16s(nt, v[hf], off, lds_addr + Gm::TILE_B + u * Gm::GS);
    }
}

// The walk over a launch's work items as every wave of a workgroup sees it; the three forms are described at
// attn_split_kernel.  Lengths and the page table are read-only for the whole launch and every index used here
// is wave-uniform: reading them through the constant address space makes these scalar loads (s_load_dword),
// which keeps them off the vector-memory counter that paces the tile loads.
enum { kItemsSplit = 0, kItemsPrefill = 1, kItemsBalanced = 2, kItemsBySize = 3 };  // (by size: kItemsSplit, the long items first)

// Prefill of a few sequences: the order in which a launch's chunks start.  A chunk costs as many tiles as it has tokens
// before its end, and the launch ends with the last one started, so the longest come first, over all sequences (every
// sequence's last chunk first, whatever the others' lengths, left a sixth of the CUs' time empty behind them: 6 sequences of
// 0..6001 cached and 333..1500 new tokens, 28/4 heads, 315 -> 272 us; 16 of 0..4000 and 64..512, 32/8 heads 338 -> 177).
// With E = end / T in whole chunks a sequence's chunks lie on the levels E, E-1, .. E-n+1, one on each; rank r is found by
// counting the chunks above a level, a lane to a sequence and one of four levels a round (a row of 16 lanes each), so that
// a round cuts the range to a quarter and the counts are sums over a row.  (A lane to a level instead, with a loop over the
// sequences, was fewer rounds and three times the instructions: 16 sequences of 1000 cached and 450..512 new tokens, 32/8
// heads, 2.4 % for the search alone where this one costs 0.2 %.)
// (A row holds 16 sequences, hence the limit.  Larger batches would gain as well: with a limit of 64, 24 / 32 / 48 sequences
// of 0..4000 tokens at 28/4 heads 269 -> 187 / 477 -> 258 / 276 -> 205 us, 24 of equal lengths 106 -> 114.)
constexpr int kRankedBatch = 16;

// A wave's lanes as the search sees them; the host has its own, for tests of the order.
struct WaveLanes {
    using Int = int;
    static __device__ __forceinline__ int lane() { return threadIdx.x & 63; }
    static __device__ __forceinline__ int lesser(int a, int b) { return min(a, b); }
    static __device__ __forceinline__ int larger(int a, int b) { return max(a, b); }
    template <class F>
    static __device__ __forceinline__ int over_row(int x, F f)  // every lane gets the value of its row of 16
    {
        x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false));  // row_ror:8, 4, 2, 1
        x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false));
        x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false));
        return f(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false));
    }
    static __device__ __forceinline__ int row_sum(int x) { return over_row(x, [](int a, int b) { return a + b; }); }
    static __device__ __forceinline__ int row_max(int x) { return over_row(x, [](int a, int b) { return max(a, b); }); }
    static __device__ __forceinline__ uint64_t less(int a, int b) { return __ballot(a < b); }
    static __device__ __forceinline__ int read(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
};

// The chunk of rank r (from 0, longest first): sequence and chunk index, false past the last.  Lane x of a row holds the
// end level and the chunk count of sequence x, both 0 for one without chunks and past the batch.
template <class Wave>
__host__ __device__ __forceinline__ bool ranked_chunk(int r, typename Wave::Int end_level, typename Wave::Int chunks, int *seq, int *chunk)
{
    using Int = typename Wave::Int;
    const Int row = Wave::lane() >> 4;
    int lo = -1, hi = Wave::read(Wave::row_max(end_level), 0), above = 0;  // more than r chunks lie above lo, `above` <= r above hi
    while (hi - lo > 1) {
        const int step = (hi - lo + 3) >> 2;
        const Int level = Wave::lesser((row + 1) * step + lo, hi);  // (the last row stands at hi)
        const Int count = Wave::row_sum(Wave::lesser(Wave::larger(end_level - level, 0), chunks));
        const int f = __builtin_ctzll(Wave::less(count, r + 1));
        if (f > 0) lo = Wave::read(level, f - 1);
        hi = Wave::read(level, f);
        above = Wave::read(count, f);
    }
    const Int down = end_level - hi;  // how far this sequence's end lies above the level
    uint64_t mask = Wave::less(down, chunks) & ~Wave::less(down, 0) & 0xffff;
    for (int k = r - above; k > 0 && mask; --k) mask &= mask - 1;
    if (!mask) return false;
    const int b = __builtin_ctzll(mask);
    *seq = b;
    *chunk = Wave::read(chunks - 1 - down, b);
    return true;
}

// Decode-mode items of different lengths: the long ones start first (decode_by_size).  A batch whose lengths only rise or only
// fall (the training mask's anchors, a queue kept sorted) shows that in a few samples, which the scalar loads of the other
// arguments' round trip bring; then the order is the batch's own, from its long end.  Otherwise, up to kRankedLens sequences
// are ranked; a larger batch starts from the end whose sequence is the longer one.  The plain order stays where the samples
// are alike: of one count of whole tiles for the 64-row kernel, within an eighth for the 32- and 16-row ones, where up to there
// the order gave nothing and its loads cost up to 2 %.
// Measured (plain -> from the long end / ranked, us per call): mask of one sequence of 4096 tokens, 256 blocks of 16, 237 -> 164 / 178
// (a ranked item waits for a vector load in front of its first tile); of 4 packed ones of 2048 (1024 items a head, a
// sawtooth) 622 -> 595 / -; of 3 of 2048, 64 blocks of 32 at 28/4 heads 154 -> 116 / 109; 128 sequences of 300..2500 in any order, 128
// rows, 180 -> 163 / 142; 100 of 100..2500, 224 rows, 113 -> 109 / 84; 200 of 50..900, 32 rows, 82 -> 78 / 71.  Above kRankedLens, 400
// sequences of 100..1500 in any order (three of them), 16 rows 245 -> 233, 239 -> 231, 235 -> 234; 64 rows 273 -> 259, 270 -> 263, 266
// -> 265; 128 rows 319 -> 290, 308 -> 296, 303 -> 293.
// Lengths nearly alike (plain -> in order -> as it is): 128 sequences at 64 rows, 1000 each 108.7 -> 109.9 -> 109.2, 1000..1031
// 108.6 -> 110.7 rising, 110.6 in any order -> 108.9, 1000..1249 in any order 121.7 -> 120.6 -> 120.3; 128 rows, 1000..1031 rising 115.4 ->
// 111.7 -> 111.2, 1000..1249 in any order 125.8 -> 122.1 -> 121.6; 16 rows, 256 of 1000..1031 in any order 182.9 -> 184.4 -> 181.4.
// A sequence's heads moved on by one from rank to rank, so that no XCD keeps to one head: no gain where
// K/V stream from memory, 1 to 5 % lost where the items of a sequence share them (mask of 4 x 2048, 60 blocks 142 -> 151).
constexpr int kOrderSamples = 6;
__host__ __device__ __forceinline__ uint32_t order_sample(int k, int batch) { return (uint32_t)(batch - 1) * (uint32_t)k / (kOrderSamples - 1); }
enum Direction { kDirUnknown, kDirAlike, kDirUp, kDirDown };
constexpr int kRankedLens = 256;

// What the samples say.  `small_counts`: a tile more or less is an order worth keeping; else a spread of an eighth.
__host__ __device__ __forceinline__ Direction direction_of(const int (&sample)[kOrderSamples], int batch, bool small_counts)
{
    int tiles[kOrderSamples];  // whole ones (bad lengths, which are checked later, only come out of order)
#pragma unroll
    for (int k = 0; k < kOrderSamples; ++k) tiles[k] = sample[k] >> 5;
    int low = tiles[0], high = tiles[0];
    bool up = true, down = true;
#pragma unroll
    for (int k = 1; k < kOrderSamples; ++k) {
        low = tiles[k] < low ? tiles[k] : low;
        high = tiles[k] > high ? tiles[k] : high;
        up = up && tiles[k - 1] <= tiles[k];
        down = down && tiles[k - 1] >= tiles[k];
    }
    if (high == low || (!small_counts && (high - low) * 8 <= high)) return kDirAlike;
    const int first = tiles[0], last = tiles[kOrderSamples - 1];
    if (batch > kRankedLens) return first < last ? kDirUp : first > last ? kDirDown : kDirAlike;
    return up ? kDirUp : down ? kDirDown : kDirUnknown;
}

// The lengths of a batch of up to kRankedLens sequences, a lane to a sequence (64 sequences a register), and the sequence of a
// rank by length in whole tiles, longest first, lower index first among equals.
struct RankedLens {
    static constexpr int REGS = kRankedLens / 64;
    int raw[REGS], tiles[REGS];
    int top;  // more than the largest number of tiles there may be

    // false when all lengths come to the same number of tiles
    __device__ __forceinline__ bool load(const AttnArgs &a)
    {
        const int lane = threadIdx.x & 63;
        // loads past the batch give 0
        const auto lens = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(a.seq_lens), 0, a.batch * 4, 0x00020000);
        top = ((a.max_seq_len + 31) >> 5) + 1;
        bool differ = false;
#pragma unroll
        for (int k = 0; k < REGS; ++k) raw[k] = __builtin_amdgcn_raw_buffer_load_b32(lens, (k * 64 + lane) * 4, 0, 0);
        const int first = (min(max(__builtin_amdgcn_readfirstlane(raw[0]), 0), a.max_seq_len) + 31) >> 5;
#pragma unroll
        for (int k = 0; k < REGS; ++k) {
            const int n = (min(max(raw[k], 0), a.max_seq_len) + 31) >> 5;
            const bool there = k * 64 + lane < a.batch;
            differ |= there && n != first;
            tiles[k] = there ? n : -1;
        }
        return __any(differ);
    }
    __device__ __forceinline__ int at_rank(int r, int *len) const
    {
        int lo = 0, hi = top, above = 0;  // more than r sequences have lo tiles or more, `above` <= r have hi or more
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            int count = 0;
#pragma unroll
            for (int k = 0; k < REGS; ++k) count += __popcll(__ballot(tiles[k] >= mid));
            if (count > r) {
                lo = mid;
            } else {
                hi = mid;
                above = count;
            }
        }
        int left = r - above, b = 0;
        *len = 0;
#pragma unroll
        for (int k = 0; k < REGS; ++k) {
            uint64_t mask = __ballot(tiles[k] == lo);
            const int n = __popcll(mask);
            if (left >= 0 && left < n) {
                for (int x = left; x > 0; --x) mask &= mask - 1;
                const int lane = __builtin_ctzll(mask);
                b = k * 64 + lane;
                *len = __builtin_amdgcn_readlane(raw[k], lane);
            }
            left -= n;
        }
        return b;
    }
};

// The NT argument of the 32-row and 16-row kernels' balanced form, which asks the call (attn_split_kernel).
constexpr int kNtAsked = 2;

#ifndef ORTHRUS_ATTN_STAGES
#define ORTHRUS_ATTN_STAGES 3
#endif
constexpr int kStages = ORTHRUS_ATTN_STAGES;  // LDS ring depth of these kernels (2..4)

template <int MODE>
struct WorkItems {
    int b, g;
    int t_begin, t_end, n_cache, n_tiles;  // cache tokens [t_begin, t_end) in n_cache tiles; n_tiles adds the in-block tile
    bool final_out;                        // this item holds every tile of its unit: write finished rows
    size_t part_slot;                      // else: index of the partial it writes
    int row0, rows_live;  // block rows of the item (prefill: first new-token index of the chunk, tokens in it)
    int pos0;             // prefill: cache position of the chunk's first token
    const const_i32 *pt_row;
    int64_t head_off;
    int bal_b, bal_g, bal_o, bal_left;  // balanced form: position in the launch's tile sequence

    // validated length of sequence x (scalar)
    __device__ __forceinline__ int seq_len(const AttnArgs &a, int x) { return checked_len(a, ((const const_i32 *)a.seq_lens)[x]); }
    __device__ __forceinline__ int checked_len(const AttnArgs &a, int L)
    {
        if (L < 0 || L > a.max_seq_len) {
            if (threadIdx.x == 0) atomicExch(a.err_word, -4);
            L = L < 0 ? 0 : a.max_seq_len;
        }
        return __builtin_amdgcn_readfirstlane(L);  // wave-uniform by construction; keeps the loop control scalar
    }

    // Finds the workgroup's share (balanced form); the others need nothing.
    __device__ __forceinline__ void start(const AttnArgs &a)
    {
        part_slot = 0;
        row0 = 0;
        rows_live = a.block_k;
        pos0 = 0;
        bal_left = 0;
        if constexpr (MODE == kItemsBalanced) {
            const int lane = threadIdx.x & 63;
            // tiles of sequence x as a lane sees it (cache tiles + the in-block tile), 0 past the batch
            auto lane_tiles = [&](int x) __attribute__((always_inline)) {
                if (x >= a.batch) return 0;
                int L = a.seq_lens[x];
                L = L < 0 ? 0 : (L > a.max_seq_len ? a.max_seq_len : L);
                return ((L + 31) >> 5) + 1;
            };
            int per_head = 0;  // tiles of one head's units
            for (int x0 = 0; x0 < a.batch; x0 += 64) {
                int n = lane_tiles(x0 + lane);
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
                per_head += n;
            }
            per_head = __builtin_amdgcn_readfirstlane(per_head);
            const int64_t total = (int64_t)per_head * a.num_kv_heads;
            const int64_t nwg = total < (int64_t)gridDim.x ? total : (int64_t)gridDim.x;
            if ((int64_t)blockIdx.x >= nwg) return;
            const int64_t c0 = (int64_t)blockIdx.x * total / nwg, c1 = ((int64_t)blockIdx.x + 1) * total / nwg;
            bal_left = __builtin_amdgcn_readfirstlane((int)(c1 - c0));
            bal_g = __builtin_amdgcn_readfirstlane((int)(c0 / per_head));
            const int r = (int)(c0 - (int64_t)bal_g * per_head);
            // the sequence whose tiles contain offset r of the head: inclusive scan over 64 sequences at a time
            int base = 0;
            for (int x0 = 0; x0 < a.batch; x0 += 64) {
                const int n = lane_tiles(x0 + lane);
                int incl = n;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int up = __shfl_up(incl, off);
                    if (lane >= off) incl += up;
                }
                const bool hit = n > 0 && base + incl - n <= r && r < base + incl;
                const uint64_t mask = __ballot(hit);
                if (mask) {
                    const int src = __builtin_ctzll(mask);
                    bal_b = x0 + src;
                    bal_o = r - (base + __shfl(incl - n, src));
                    break;
                }
                base += __shfl(incl, 63);
            }
            bal_b = __builtin_amdgcn_readfirstlane(bal_b);
            bal_o = __builtin_amdgcn_readfirstlane(bal_o);
        }
    }

    // Fixed splits, the items that are long first (decode_by_size): finds b, g, the split and the length.  The items of a sequence
    // follow each other, its heads fastest; with lengths alike, the plain order.
    __device__ __forceinline__ void find_by_size(const AttnArgs &a, bool small_counts, int *split, int *len)
    {
        // what the batch's address and size alone lead to, in the round trip that the other arguments take: samples of the
        // batch, and the length that the plain order names
        const const_i32 *lens = (const const_i32 *)a.seq_lens;
        const int last = a.batch - 1;
        int sample[kOrderSamples];
#pragma unroll
        for (int k = 0; k < kOrderSamples; ++k) sample[k] = lens[order_sample(k, a.batch)];
        *len = lens[b];
        const Direction dir = direction_of(sample, a.batch, small_counts);
        const unsigned heads = (unsigned)a.num_kv_heads, splits = (unsigned)a.num_splits;
        g = (int)(blockIdx.x / ((unsigned)a.batch * splits));
        *split = (int)(blockIdx.x / (unsigned)a.batch % splits);
        if (dir != kDirAlike) {
            const int rank = (int)(blockIdx.x / (heads * splits)), item = (int)(blockIdx.x % (heads * splits));
            RankedLens ranked;
            bool in_turn = true;
            if (dir == kDirUnknown) {
                in_turn = ranked.load(a);
                if (in_turn) b = ranked.at_rank(rank, len);
            } else {
                b = dir == kDirUp ? last - rank : rank;
                *len = lens[b];
            }
            if (in_turn) {
                g = item % (int)heads;
                *split = item / (int)heads;
            }
        }
        *len = checked_len(a, *len);
    }

    // Opens the next work item; false when the workgroup has none (left).
    __device__ __forceinline__ bool open(const AttnArgs &a, bool small_counts = false)
    {
        if constexpr (MODE == kItemsBalanced) {
            if (bal_left <= 0) return false;
            b = bal_b;
            g = bal_g;
            const int L = seq_len(a, b);
            const int nc = (L + 31) >> 5;                    // cache tiles of the unit; the in-block tile is tile nc
            const int take = min(nc + 1 - bal_o, bal_left);  // tiles of this segment
            const bool has_blk = bal_o + take == nc + 1;
            // (everything here is wave-uniform; readfirstlane keeps it in scalar registers)
            n_tiles = __builtin_amdgcn_readfirstlane(take);
            n_cache = has_blk ? n_tiles - 1 : n_tiles;
            t_begin = __builtin_amdgcn_readfirstlane(bal_o * 32);
            t_end = min(L, t_begin + n_cache * 32);
            final_out = bal_o == 0 && has_blk;
            part_slot = (size_t)(blockIdx.x * 2u + (bal_o == 0 ? 1u : 0u));
            bal_left = __builtin_amdgcn_readfirstlane(bal_left - take);
            bal_o = 0;
            int nb = bal_b + 1, ng = bal_g;
            if (nb == a.batch) {
                nb = 0;
                ++ng;
            }
            bal_b = __builtin_amdgcn_readfirstlane(nb);
            bal_g = __builtin_amdgcn_readfirstlane(ng);
        } else {
            // Workgroup id -> work item.  Consecutive workgroup ids go to different XCDs.
            // Decode: the sequence index is fastest and the KV head slowest.  A head's rows sit at a fixed offset
            // inside every page, so an order that ties XCD k to head k makes each XCD hammer its own subset of the
            // HBM channels and the XCDs finish far apart.  (By size the heads are fastest all the same: with lengths that differ,
            // what the order gives is more, and sequences of the 64-row kernel gain 4 % even where they hardly differ.)
            // Prefill: the sequence is fastest, then the head, then the chunk, every sequence's last (the one with the
            // most cache tokens) first.  Ranked prefill: the head is fastest, then the chunk's rank; a chunk's heads
            // are alike in length.
            b = (int)(blockIdx.x % (unsigned)a.batch);
            int split;
            if constexpr (MODE == kItemsPrefill) {
                // lengths as the append kernel left them: validated, 0 new tokens on a capacity error
                g = (int)((blockIdx.x / (unsigned)a.batch) % (unsigned)a.num_kv_heads);
                int L0, n_new, chunk = -1;
                bool alike = true;
                if (a.ranked) {
                    const int x = threadIdx.x & 15, y = min(x, a.batch - 1);
                    const int lane_old = a.old_lens[y], lane_new = a.new_lens[y];
                    L0 = __builtin_amdgcn_readfirstlane(lane_old);
                    n_new = __builtin_amdgcn_readfirstlane(lane_new);
                    alike = !__any(lane_old != L0 || lane_new != n_new);  // all of one length: the plain order is the ranked one
                    if (!alike) {
                        g = (int)(blockIdx.x % (unsigned)a.num_kv_heads);
                        const int chunks = x < a.batch ? (lane_new + a.chunk_tokens - 1) / a.chunk_tokens : 0;
                        const int end_level = chunks > 0 ? (lane_old + lane_new) / a.chunk_tokens : 0;
                        if (!ranked_chunk<WaveLanes>((int)(blockIdx.x / (unsigned)a.num_kv_heads), end_level, chunks, &b, &chunk))
                            return false;
                        L0 = __builtin_amdgcn_readlane(lane_old, b);
                        n_new = __builtin_amdgcn_readlane(lane_new, b);
                    }
                } else {
                    L0 = __builtin_amdgcn_readfirstlane(((const const_i32 *)a.old_lens)[b]);
                    n_new = __builtin_amdgcn_readfirstlane(((const const_i32 *)a.new_lens)[b]);
                }
                if (alike) {
                    split = (int)(blockIdx.x / ((unsigned)a.batch * (unsigned)a.num_kv_heads));
                    chunk = (n_new + a.chunk_tokens - 1) / a.chunk_tokens - 1 - split;
                    if (chunk < 0) return false;
                }
                // this launch reads the recorded lengths only, so the sequence's first chunk may bump the live one
                if (chunk == 0 && g == 0 && threadIdx.x == 0) a.seq_lens_out[b] = L0 + n_new;
                row0 = chunk * a.chunk_tokens;
                rows_live = min(a.chunk_tokens, n_new - row0);
                pos0 = L0 + row0;
                t_begin = 0;
                t_end = pos0 + rows_live;  // everything up to the chunk's last token
                n_cache = (t_end + 31) >> 5;
                n_tiles = n_cache;
                final_out = true;
            } else {
                int L;
                if constexpr (MODE == kItemsBySize) {
                    find_by_size(a, small_counts, &split, &L);
                } else {
                    split = (int)((blockIdx.x / (unsigned)a.batch) % (unsigned)a.num_splits);
                    g = (int)(blockIdx.x / ((unsigned)a.batch * (unsigned)a.num_splits));
                    L = seq_len(a, b);
                }
                return take(a, split, L);
            }
        }
        point(a);
        return true;
    }

    // Piece `split` of unit (b, g), whose length is L; false when nothing falls in it.
    __device__ __forceinline__ bool take(const AttnArgs &a, int split, int L)
    {
        // The sequence's own length, not the host's bound on it, is cut into num_splits pieces:
        // they stay equal however loose the bound is (it only sized the grid), e.g. when a
        // decode loop bumps it by K per step without reading back.
        const SplitCut cut = split_cut(L, a.num_splits, split);
        if (cut.count == 0) return false;  // fewer tiles than splits: nothing falls in this one
        n_tiles = __builtin_amdgcn_readfirstlane(cut.count);
        n_cache = split == cut.live - 1 ? n_tiles - 1 : n_tiles;  // the last piece ends with the in-block tile
        t_begin = __builtin_amdgcn_readfirstlane(cut.first * 32);
        t_end = min(L, t_begin + n_cache * 32);
        final_out = a.num_splits == 1;
        part_slot = ((size_t)b * a.num_kv_heads + g) * a.num_splits + split;
        point(a);
        return true;
    }

    __device__ __forceinline__ void point(const AttnArgs &a)
    {
        pt_row = (const const_i32 *)(a.page_table + (int64_t)b * a.max_pages_per_seq);
        head_off = (int64_t)g * a.stride_head;
    }
};

// Launch of one of a call's two kernels (kind 0: split, 1: combine), with its timing events attached when wanted.
template <class Kern>
inline hipError_t launch_timed(Kern kern, dim3 grid, dim3 block, size_t lds, const AttnArgs &a, hipStream_t stream,
                               AttnLaunchEvents *ev, int kind)
{
    if (ev && ev->on) {
        hipExtLaunchKernelGGL(kern, grid, block, lds, stream, ev->start[kind], ev->stop[kind], 0, ATTN_FIRST_VALUES(a), a);
        ev->used[kind] = true;
    } else {
        hipLaunchKernelGGL(kern, grid, block, lds, stream, ATTN_FIRST_VALUES(a), a);
    }
    return hipGetLastError();
}

// The compute wave of a call of at most 16 rows (orthrus_attn_forms.hip; named by the body that the kernels share).
template <int D, int NS, int MODE, int NT>
__device__ void thin_rows(const AttnArgs &a, WorkItems<MODE> it, uint32_t smem_lds);

}  // namespace orthrus
