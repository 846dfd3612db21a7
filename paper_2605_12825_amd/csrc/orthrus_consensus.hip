// Greedy consensus and in-place commit for the Orthrus decode step on gfx950 (Section 3.3,
// "Architectural Consensus Mechanism", Eq. 8; Fig. 2(b): accepted tokens' KV appended to the
// shared cache).
//
//   argmax_partial_kernel  grid (row * chunks + chunk): each workgroup scans one chunk of one logits
//                          row with 16-byte loads and reduces (value, index) through wavefront
//                          shuffles; one (value, index) pair per chunk goes to the workspace, with a mark when
//                          the index is the row's draft.
//   accept_commit_kernel   grid (sequence, layer): the four waves finish the K row argmaxes (chunk pairs
//                          spread over the lanes, wavefront-shuffle reduction), the first wave finds the
//                          accepted prefix from the marks with a wavefront ballot and checks that the appended positions
//                          are mapped; then the workgroup copies its layer's appended K/V rows into their
//                          pages.  The workgroup of layer 0 writes tokens and lengths.  (Every layer's
//                          workgroup repeats the few microseconds of the decision: a third launch that copies
//                          by it cost 4 to 7 us.  It reads nothing that layer 0's workgroup writes, drafts
//                          included: out_tokens may be draft_tokens.)
//   commit_kernel          grid (sequence, layer): the copy as a launch of its own, for many (sequence, layer)
//                          pairs (kCopyApart); accept_commit_kernel then has grid (sequence).
// (A single-launch variant in which the last-arriving workgroup of a sequence finishes the job was
// measured and dropped: the device-scope release/acquire fences it needs per workgroup cost far
// more than the second launch.)
//
// Order among candidates: a NaN outranks every number, larger values outrank smaller ones, and
// among equals the smaller index wins; this is a total order, so the result does not depend on
// how the scan is split.
#include "orthrus_internal.h"

#include <mutex>

namespace orthrus {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---- device-resident scratch of the allocation-free entry point (orthrus_consensus_commit_noalloc)
// One fixed array per GPU, held until the process ends; it takes the place of the caller's workspace
// (chunk argmax pairs and the per-sequence commit record).  Every entry it uses is written by the
// call's first kernels before anything reads it, so nothing has to start at zero.  Host code never
// passes the array's name to a kernel: the name is only a handle for hipGetSymbolAddress, and each
// device has its own copy at its own address, looked up once with that device current.
constexpr size_t kScratchBytes = (size_t)1 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mutex;

size_t consensus_scratch_bytes() { return kScratchBytes; }

hipError_t consensus_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return hipSuccess;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));  // the current device's copy
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void *consensus_scratch(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[device];
}

constexpr int kChunkElems = 8192;  // floats per (row, chunk) workgroup: 32 KiB
int consensus_chunk_elems() { return kChunkElems; }

// true if candidate (v1, i1) outranks (v2, i2)
__device__ __forceinline__ bool outranks(float v1, uint32_t i1, float v2, uint32_t i2)
{
    const bool n1 = v1 != v1, n2 = v2 != v2;
    if (n1 || n2) return (n1 && n2) ? (i1 < i2) : n1;
    return v1 > v2 || (v1 == v2 && i1 < i2);
}

// update for a candidate known to sit at a larger index than the current best
__device__ __forceinline__ void take_later(float v, uint32_t i, float &bv, uint32_t &bi)
{
    if (!(bv != bv) && ((v != v) || v > bv)) { bv = v; bi = i; }
}

__device__ __forceinline__ void wave_best(float &bv, uint32_t &bi)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off);
        const uint32_t oi = (uint32_t)__shfl_xor((int)bi, off);
        if (outranks(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
}

__global__ void __launch_bounds__(256) argmax_partial_kernel(const ConsensusArgs a)
{
    const int row = blockIdx.x / a.chunks, chunk = blockIdx.x - row * a.chunks;
    const int tid = threadIdx.x;
    const float *base = a.ar_logits + (int64_t)row * a.vocab;
    const int begin = chunk * a.chunk_elems;
    const int end = min(a.vocab, begin + a.chunk_elems);
    float bv = -INFINITY;
    uint32_t bi = 0x7fffffff;
    const int draft = tid == 0 ? a.draft_tokens[row] : -1;
    if (a.do_commit && tid == 0 && chunk == 0 && row % a.block_k == 0) commit_snapshot(a, row / a.block_k);
    // The 16-byte aligned middle of the chunk, all of a thread's loads before the first comparison (kChunkElems / 1024
    // = 8 of 16 bytes), and up to three elements on either side of it (a row starts anywhere when the vocabulary is
    // not a multiple of four; element by element such a scan took three times as long).
    const int head = min((int)((0 - ((uintptr_t)(base + begin) >> 2)) & 3), end - begin);
    const int mid = begin + head, nvec = (end - mid) >> 2, tail = mid + 4 * nvec;
    constexpr int NL = kChunkElems / (256 * 4);
    float4 x[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int v = u * 256 + tid;
        x[u] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (v < nvec) {  // read once, never again: do not let the row displace anything in the caches
            const f32x4 t = __builtin_nontemporal_load((const f32x4 *)(base + mid) + v);
            x[u] = make_float4(t[0], t[1], t[2], t[3]);
        }
    }
    const int edge = tid < 4 ? (tid < head ? begin + tid : end) : tid < 8 ? tail + tid - 4 : end;
    const float xe = edge < end ? base[edge] : -INFINITY;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int i = mid + (u * 256 + tid) * 4;
        if (u * 256 + tid < nvec) {
            if (bi == 0x7fffffff) { bv = x[u].x; bi = i; } else take_later(x[u].x, i, bv, bi);
            take_later(x[u].y, i + 1, bv, bi);
            take_later(x[u].z, i + 2, bv, bi);
            take_later(x[u].w, i + 3, bv, bi);
        }
    }
    if (edge < end && outranks(xe, edge, bv, bi)) { bv = xe; bi = edge; }
    wave_best(bv, bi);
    __shared__ float sv[4];
    __shared__ uint32_t si[4];
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < 4; ++w)
            if (outranks(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
        a.part_val[(int64_t)row * a.chunks + chunk] = bv;
        a.part_idx[(int64_t)row * a.chunks + chunk] = bi << 1 | (bi == (uint32_t)draft ? 1u : 0u);
    }
}

__global__ void __launch_bounds__(256) accept_commit_kernel(const ConsensusArgs a)
{
    const int b = blockIdx.x, layer = blockIdx.y, tid = threadIdx.x;
    const bool lead = layer == 0;
    const int K = a.block_k;
    __shared__ int s_L, s_m;
    __shared__ uint32_t s_am[32];  // index << 1 | mark
    __shared__ int s_pg[32];
    const int wave = tid >> 6, lane = tid & 63;
    // ---- loads that do not depend on the argmaxes go out first (first wave): the length and the page ids of the K
    // positions that may be appended
    CommitProbe probe = {0, -1};
    if (wave == 0 && a.do_commit) probe = commit_probe(a, b, lane);
    // ---- row argmaxes: wave w finishes rows w, w+4, ...; a lane takes the chunk pairs lane, lane+64, ...
    // All loads of a wave's rows go out before the first reduction, so the phase costs one memory round
    // trip, not one per chunk.  A lane without a chunk holds (-inf, UINT_MAX), which every real pair outranks.
    {
        constexpr int kRowsPerWave = 8;  // block_k <= 32 rows over 4 waves
        float bv[kRowsPerWave];
        uint32_t bi[kRowsPerWave];
#pragma unroll
        for (int u = 0; u < kRowsPerWave; ++u) {
            const int k = wave + 4 * u;
            bv[u] = -INFINITY;
            bi[u] = 0xffffffffu;
            if (k < K) {
                const int64_t r = ((int64_t)b * K + k) * a.chunks;
                for (int ch = lane; ch < a.chunks; ch += 64) {
                    const float v = a.part_val[r + ch];
                    const uint32_t i = a.part_idx[r + ch];
                    if (outranks(v, i, bv[u], bi[u])) { bv[u] = v; bi[u] = i; }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kRowsPerWave; ++u) {
            const int k = wave + 4 * u;
            if (k < K) {  // wave-uniform
                wave_best(bv[u], bi[u]);
                if (lane == 0) s_am[k] = bi[u];
            }
        }
    }
    __syncthreads();
    // ---- accept: the first wave, lane k < K owns block row k of sequence b
    if (wave == 0) {
        int am = -1;
        bool match = false;
        if (lane < K) {
            am = (int)(s_am[lane] >> 1);
            match = s_am[lane] & 1u;
        }
        // accepted prefix = run of matching rows starting at row 0
        const unsigned long long mism = ~__ballot(match);           // lanes >= K never match
        const int n_acc = mism ? __ffsll((long long)mism) - 1 : 64;  // first mismatching row (<= K)
        const int m = min(n_acc + 1, K);
        if (lead && lane < K) a.out_tokens[(int64_t)b * K + lane] = lane < m ? am : -1;
        const int anchor = __shfl(am, m - 1);
        int committed = m;
        if (a.do_commit) {
            committed = commit_decide(a, b, lane, m, probe, lead);
            if (lane < K) s_pg[lane] = probe.pg;
        }
        if (lane == 0) {
            if (lead) {
                a.accept_len[b] = n_acc;
                a.num_committed[b] = committed;
                a.next_anchor[b] = anchor;
            }
            s_L = probe.L;
            s_m = a.do_commit && !a.copy_apart ? committed : 0;
            if (a.copy_apart) a.decided[b] = committed;
        }
    }
    __syncthreads();
    // ---- commit: this workgroup's layer
    if (s_m > 0) append_rows(a, b, layer, s_L, s_m, tid, 256, s_pg);
}

// The same copy as its own launch.
__global__ void __launch_bounds__(256) commit_kernel(const ConsensusArgs a)
{
    const int b = blockIdx.x, layer = blockIdx.y;
    const int m = a.decided[b];
    if (m > 0) append_rows(a, b, layer, a.commit_info[b], m, threadIdx.x, 256);
}

// From this many (sequence, layer) pairs on, repeating the decision in each costs more than a third launch: 64 x 16 rows,
// 36 layers (2304 pairs) 42 us against 44 with the copy apart; 80 x 16, 36 layers (2880) 47 against 45; 64 x 32, 48 layers
// 75 against 68; 64 x 32, 64 layers 91 against 77; 512 x 16, 36 layers 216 against 189.  (Several layers to a workgroup,
// one after the other: 86 us at 64 x 32 x 64, 156 at 256 x 16 x 36 where one launch of a workgroup each takes 123.)
constexpr int kCopyApart = 2560;

hipError_t launch_consensus(ConsensusArgs a, hipStream_t stream)
{
    if (a.batch == 0) return hipSuccess;
    a.copy_apart = a.do_commit && (int64_t)a.batch * a.num_layers >= kCopyApart;
    dim3 g1((unsigned)a.chunks * (unsigned)(a.batch * a.block_k));
    hipLaunchKernelGGL(argmax_partial_kernel, g1, dim3(256), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(accept_commit_kernel, dim3(a.batch, a.do_commit && !a.copy_apart ? a.num_layers : 1), dim3(256), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess || !a.copy_apart) return e;
    hipLaunchKernelGGL(commit_kernel, dim3(a.batch, a.num_layers), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace orthrus
