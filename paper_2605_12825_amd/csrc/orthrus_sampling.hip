// Lossless consensus for temperature T > 0 on gfx950 (Section 3.3: exact rejection sampling after the
// speculative-sampling rule the paper cites): with p_k = softmax(ar_logits[k] / T) and
// q_k = softmax(diff_logits[k] / T), draft x of row k is kept iff accept_u[k] * q_k(x) < p_k(x); at the
// first row j that is not kept the emitted token is argmax_v [ log max(0, p_j - q_j)(v) + gumbel(v) ]
// (a draw from the normalised positive part of p_j - q_j; from p_j if that part is empty).  All random
// numbers are inputs, so the step is a deterministic function of its arguments.
//
//   lse_partial_kernel      grid (row * chunks + chunk): (max, sum of exp) of both scaled logit rows
//                           over one 8192-element chunk, 16-byte loads, wavefront shuffles.
//   draw_partial_kernel     grid (draw chunk, sequence): every workgroup re-derives the K keep decisions of
//                           its sequence from the chunk pairs (same code, same order => same answer
//                           everywhere), and if a row j < K was rejected scans its 2048-element piece of row
//                           j for the two candidate maxima.  The first one records j; each raises a
//                           draw key to its own (a total order: the result does not depend on timing).
//   sample_commit_kernel    grid (sequence, layer): the workgroup of layer 0 takes the largest draw key and
//                           writes the outputs, every layer's workgroup commits its layer's kept rows.  Only
//                           layer 0's reads the drafts, before it writes the tokens: out_tokens may be
//                           draft_tokens.
// The two small kernels are chains of memory round trips and exponentials.  Eight threads share a row's chunk pairs
// and the draw's pieces are small, so that a batch of one fills 63 workgroups instead of 16 with four times fewer
// exponentials per thread (batch 1, K = 16, V = 128256: 14.2 + 9.0 -> 7.5 + 4.1 us; batch 8, K = 32, V = 151936: 16.9 +
// 11.3 -> 9.9 + 4.9).
#include "orthrus_internal.h"

namespace orthrus {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kSChunk = 8192;
constexpr int kDrawChunk = 2048;
int draw_chunk_elems() { return kDrawChunk; }

__device__ __forceinline__ void lse_merge(float &m, float &s, float m2, float s2)
{
    const float mn = fmaxf(m, m2);
    if (mn == -INFINITY) { m = mn; s = 0.f; return; }
    s = s * expf(m - mn) + s2 * expf(m2 - mn);
    m = mn;
}

__global__ void __launch_bounds__(256) lse_partial_kernel(const SamplingArgs a)
{
    const int chunks = a.c.chunks, V = a.c.vocab;
    const int row = blockIdx.x / chunks, chunk = blockIdx.x - row * chunks;
    const int tid = threadIdx.x;
    const float *pr = a.c.ar_logits + (int64_t)row * V;
    const float *qr = a.diff_logits + (int64_t)row * V;
    const int begin = chunk * kSChunk, end = min(V, begin + kSChunk);
    const float it = a.inv_temperature;
    if (row % a.c.block_k == 0) {
        const int b = row / a.c.block_k;
        if (tid < 2) a.draw_key[((int64_t)b * chunks + chunk) * 2 + tid] = 0;
        if (a.c.do_commit && tid == 0 && chunk == 0) commit_snapshot(a.c, b);
    }
    constexpr int PER = kSChunk / 256;  // 32 values per thread and row
    float xp[PER], xq[PER];
    // 16-byte loads of the aligned middle, and up to three elements on either side of it (a row starts anywhere when
    // the vocabulary is not a multiple of four), if both logit sets are aligned alike; else element by element.
    float xpe = -INFINITY, xqe = -INFINITY;
    const int skew = (int)((0 - ((uintptr_t)(pr + begin) >> 2)) & 3);
    if (skew == (int)((0 - ((uintptr_t)(qr + begin) >> 2)) & 3)) {
        const int head = min(skew, end - begin), mid = begin + head, nvec = (end - mid) >> 2, tail = mid + 4 * nvec;
#pragma unroll
        for (int u = 0; u < PER / 4; ++u) {
            const int v = u * 256 + tid;
            float4 vp = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY), vq = vp;
            if (v < nvec) {  // one pass over both logit sets: loads that do not displace anything in the caches
                const f32x4 tp = __builtin_nontemporal_load((const f32x4 *)(pr + mid) + v);
                const f32x4 tq = __builtin_nontemporal_load((const f32x4 *)(qr + mid) + v);
                vp = make_float4(tp[0], tp[1], tp[2], tp[3]);
                vq = make_float4(tq[0], tq[1], tq[2], tq[3]);
            }
            xp[4 * u] = vp.x; xp[4 * u + 1] = vp.y; xp[4 * u + 2] = vp.z; xp[4 * u + 3] = vp.w;
            xq[4 * u] = vq.x; xq[4 * u + 1] = vq.y; xq[4 * u + 2] = vq.z; xq[4 * u + 3] = vq.w;
        }
        const int edge = tid < 4 ? (tid < head ? begin + tid : end) : tid < 8 ? tail + tid - 4 : end;
        if (edge < end) {
            xpe = pr[edge];
            xqe = qr[edge];
        }
    } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = begin + u * 256 + tid;
            xp[u] = i < end ? pr[i] : -INFINITY;
            xq[u] = i < end ? qr[i] : -INFINITY;
        }
    }
    // Per thread: maximum of the raw logits (1/T > 0 keeps the order), then the sum of
    // exp((x - max) / T) as exp2 of one fused multiply-add per element.  Entries past the end are
    // -inf and add exp2(-inf) = 0; a thread that saw nothing but -inf keeps (max, sum) = (-inf, 0).
    float rp = xpe, rq = xqe;
#pragma unroll
    for (int u = 0; u < PER; ++u) { rp = fmaxf(rp, xp[u]); rq = fmaxf(rq, xq[u]); }
    const float c2 = it * 1.4426950408889634f;  // log2(e) / T
    const float bp = rp == -INFINITY ? 0.f : -rp * c2, bq = rq == -INFINITY ? 0.f : -rq * c2;
    float sp = __builtin_amdgcn_exp2f(__builtin_fmaf(xpe, c2, bp)), sq = __builtin_amdgcn_exp2f(__builtin_fmaf(xqe, c2, bq));
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        sp += __builtin_amdgcn_exp2f(__builtin_fmaf(xp[u], c2, bp));
        sq += __builtin_amdgcn_exp2f(__builtin_fmaf(xq[u], c2, bq));
    }
    float mp = rp * it, mq = rq * it;  // maxima of the scaled logits (natural-log domain from here on)
    // wavefront, then workgroup merge in a fixed order
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lse_merge(mp, sp, __shfl_xor(mp, off), __shfl_xor(sp, off));
        lse_merge(mq, sq, __shfl_xor(mq, off), __shfl_xor(sq, off));
    }
    __shared__ float4 sh[4];
    if ((tid & 63) == 0) sh[tid >> 6] = make_float4(mp, sp, mq, sq);
    __syncthreads();
    if (tid == 0) {
        float4 r = sh[0];
#pragma unroll
        for (int w = 1; w < 4; ++w) { lse_merge(r.x, r.y, sh[w].x, sh[w].y); lse_merge(r.z, r.w, sh[w].z, sh[w].w); }
        a.lse_part[(int64_t)row * chunks + chunk] = r;
    }
}

// Keep decisions of sequence b, made by the whole workgroup: eight threads per row merge its chunk pairs (a fixed tree:
// every eighth chunk in order, then by shuffles).  Returns the first row that is not kept (K if none) and, for that
// row, the two log-sum-exps.  Contains barriers.
__device__ __forceinline__ int first_rejected(const SamplingArgs &a, int b, int tid, float &lsep_j, float &lseq_j)
{
    const int K = a.c.block_k, V = a.c.vocab, chunks = a.c.chunks;
    const int k = tid >> 3, sub = tid & 7;
    __shared__ int s_keep[32];
    __shared__ float2 s_lse[32];
    if (k < K) {
        const int64_t row = (int64_t)b * K + k;
        const int x = a.c.draft_tokens[row];
        const float4 *part = a.lse_part + row * chunks;
        float4 r = make_float4(-INFINITY, 0.f, -INFINITY, 0.f);
        for (int c0 = sub; c0 < chunks; c0 += 32) {  // four loads in flight
            float4 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = c0 + 8 * u < chunks ? part[c0 + 8 * u] : make_float4(-INFINITY, 0.f, -INFINITY, 0.f);
            const float mp = fmaxf(fmaxf(fmaxf(t[0].x, t[1].x), fmaxf(t[2].x, t[3].x)), r.x);
            const float mq = fmaxf(fmaxf(fmaxf(t[0].z, t[1].z), fmaxf(t[2].z, t[3].z)), r.z);
            float sp = mp == -INFINITY ? 0.f : r.y * expf(r.x - mp), sq = mq == -INFINITY ? 0.f : r.w * expf(r.z - mq);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (mp != -INFINITY) sp += t[u].y * expf(t[u].x - mp);
                if (mq != -INFINITY) sq += t[u].w * expf(t[u].z - mq);
            }
            r = make_float4(mp, sp, mq, sq);
        }
        const bool valid = x >= 0 && x < V;
        const float ap = valid ? a.c.ar_logits[row * V + x] : 0.f, aq = valid ? a.diff_logits[row * V + x] : 0.f;
        const float u01 = a.accept_u[row];
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            lse_merge(r.x, r.y, __shfl_xor(r.x, off), __shfl_xor(r.y, off));
            lse_merge(r.z, r.w, __shfl_xor(r.z, off), __shfl_xor(r.w, off));
        }
        const float lsep = r.x + logf(r.y), lseq = r.z + logf(r.w);
        if (sub == 0) {
            s_keep[k] = valid && u01 * expf(aq * a.inv_temperature - lseq) < expf(ap * a.inv_temperature - lsep);
            s_lse[k] = make_float2(lsep, lseq);
        }
    }
    __syncthreads();
    const int lane = tid & 63;
    const unsigned long long rej = ~__ballot(lane >= K || s_keep[lane < K ? lane : 0]);
    const int j = rej ? __ffsll((long long)rej) - 1 : K;
    const float2 l = s_lse[j < K ? j : 0];
    lsep_j = l.x;
    lseq_j = l.y;
    return j;
}

__device__ __forceinline__ bool better_score(float v1, int i1, float v2, int i2)
{
    return v1 > v2 || (v1 == v2 && i1 < i2);
}

// A candidate of the draw as one number that orders like (among p > q or not, score, smaller index first).  0 is below
// every candidate and reads as index INT_MAX.  (One such key a sequence for all pieces: 69 instead of 66 us at batch 8.)
__device__ __forceinline__ unsigned long long draw_key_of(bool positive, float score, int index)
{
    uint32_t u = __float_as_uint(score + 0.f);  // (-0 counts as 0)
    u = u >> 31 ? ~u : u | 0x80000000u;
    return (unsigned long long)positive << 63 | (unsigned long long)u << 31 | (~(uint32_t)index & 0x7fffffffu);
}

__global__ void __launch_bounds__(256) draw_partial_kernel(const SamplingArgs a)
{
    const int chunk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int K = a.c.block_k, V = a.c.vocab;
    float lsep, lseq;
    const int j = first_rejected(a, b, tid, lsep, lseq);
    if (chunk == 0 && tid == 0) a.c.decided[b] = j;
    if (j >= K) return;  // every draft kept: nothing to draw
    const float it = a.inv_temperature;
    const float *pr = a.c.ar_logits + ((int64_t)b * K + j) * V;
    const float *qr = a.diff_logits + ((int64_t)b * K + j) * V;
    const float *gr = a.gumbel + (int64_t)b * V;
    const int begin = chunk * kDrawChunk, end = min(V, begin + kDrawChunk);
    float bp = -INFINITY, ba = -INFINITY;   // best among p > q, best of log p + g
    int ip = 0x7fffffff, ia = 0x7fffffff;
    auto visit = [&](int i, float xp, float xq, float g) __attribute__((always_inline)) {
        const float lp = xp * it - lsep, lq = xq * it - lseq;
        const float r = expf(lp) - expf(lq);
        if (r > 0.f) {
            const float sc = logf(r) + g;
            if (better_score(sc, i, bp, ip)) { bp = sc; ip = i; }
        }
        const float sa = lp + g;
        if (better_score(sa, i, ba, ia)) { ba = sa; ia = i; }
    };
    const bool vec_ok = ((V & 3) == 0) &&
                        (((((uintptr_t)a.c.ar_logits) | ((uintptr_t)a.diff_logits) | ((uintptr_t)a.gumbel)) & 15) == 0);
    if (vec_ok) {
        // all of a thread's loads of the chunk go out before the first score is formed
        constexpr int NL = kDrawChunk / (256 * 4);
        float4 vp[NL], vq[NL], vg[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int i = begin + (u * 256 + tid) * 4;
            vp[u] = vq[u] = vg[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i < end) {
                vp[u] = *(const float4 *)(pr + i);
                vq[u] = *(const float4 *)(qr + i);
                vg[u] = *(const float4 *)(gr + i);
            }
        }
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int i = begin + (u * 256 + tid) * 4;
            if (i < end) {  // indices ascend within a thread, as in the scalar loop
                visit(i, vp[u].x, vq[u].x, vg[u].x);
                visit(i + 1, vp[u].y, vq[u].y, vg[u].y);
                visit(i + 2, vp[u].z, vq[u].z, vg[u].z);
                visit(i + 3, vp[u].w, vq[u].w, vg[u].w);
            }
        }
    } else {
        constexpr int NS = kDrawChunk / 256;
        float vp[NS], vq[NS], vg[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int i = begin + u * 256 + tid;
            vp[u] = vq[u] = vg[u] = 0.f;
            if (i < end) { vp[u] = pr[i]; vq[u] = qr[i]; vg[u] = gr[i]; }
        }
#pragma unroll
        for (int u = 0; u < NS; ++u)
            if (begin + u * 256 + tid < end) visit(begin + u * 256 + tid, vp[u], vq[u], vg[u]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float op = __shfl_xor(bp, off), oa = __shfl_xor(ba, off);
        const int jp = __shfl_xor(ip, off), ja = __shfl_xor(ia, off);
        if (better_score(op, jp, bp, ip)) { bp = op; ip = jp; }
        if (better_score(oa, ja, ba, ia)) { ba = oa; ia = ja; }
    }
    __shared__ float4 sh[4];
    if ((tid & 63) == 0) sh[tid >> 6] = make_float4(bp, __int_as_float(ip), ba, __int_as_float(ia));
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            if (better_score(sh[w].x, __float_as_int(sh[w].y), bp, ip)) { bp = sh[w].x; ip = __float_as_int(sh[w].y); }
            if (better_score(sh[w].z, __float_as_int(sh[w].w), ba, ia)) { ba = sh[w].z; ia = __float_as_int(sh[w].w); }
        }
        const int keys = 2 * a.c.chunks;  // (at most 4 * chunks pieces)
        unsigned long long *key = a.draw_key + (int64_t)b * keys + (chunk < keys ? chunk : chunk - keys);
        if (ip != 0x7fffffff) atomicMax(key, draw_key_of(true, bp, ip));
        else if (ia != 0x7fffffff) atomicMax(key, draw_key_of(false, ba, ia));
    }
}

__global__ void __launch_bounds__(256) sample_commit_kernel(const SamplingArgs a)
{
    const ConsensusArgs &c = a.c;
    const int b = blockIdx.x, layer = blockIdx.y, tid = threadIdx.x;
    const bool lead = layer == 0;
    const int K = c.block_k;
    __shared__ int s_L, s_m;
    __shared__ int s_pg[32];
    if (tid < 64) {
        const int lane = tid;
        const int j = c.decided[b];
        CommitProbe probe = {0, -1};
        if (c.do_commit) probe = commit_probe(c, b, lane);
        const int m = min(j + 1, K);
        if (lead) {
            unsigned long long key = 0;
            for (int d = lane; d < 2 * c.chunks; d += 64) key = max(key, a.draw_key[(int64_t)b * 2 * c.chunks + d]);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) key = max(key, (unsigned long long)__shfl_xor(key, off));
            const int repl = (int)(~(uint32_t)key & 0x7fffffffu);
            if (lane < K) {
                int t = -1;
                if (lane < j) t = c.draft_tokens[(int64_t)b * K + lane];
                else if (lane == j) t = repl;
                c.out_tokens[(int64_t)b * K + lane] = t;
            }
            if (lane == 0) {
                c.accept_len[b] = j;
                c.next_anchor[b] = j < K ? repl : c.draft_tokens[(int64_t)b * K + K - 1];
            }
        }
        int committed = m;
        if (c.do_commit) {
            committed = commit_decide(c, b, lane, m, probe, lead);
            if (lane < K) s_pg[lane] = probe.pg;
        }
        if (lane == 0) {
            if (lead) c.num_committed[b] = committed;
            s_L = probe.L;
            s_m = c.do_commit ? committed : 0;
        }
    }
    __syncthreads();
    if (s_m > 0) append_rows(c, b, layer, s_L, s_m, tid, 256, s_pg);
}

hipError_t launch_sampling_consensus(const SamplingArgs &a, hipStream_t stream)
{
    const ConsensusArgs &c = a.c;
    if (c.batch == 0) return hipSuccess;
    hipLaunchKernelGGL(lse_partial_kernel, dim3((unsigned)c.chunks * (unsigned)(c.batch * c.block_k)), dim3(256), 0,
                       stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(draw_partial_kernel, dim3(a.draw_chunks, c.batch), dim3(256), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sample_commit_kernel, dim3(c.batch, c.do_commit ? c.num_layers : 1), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace orthrus
