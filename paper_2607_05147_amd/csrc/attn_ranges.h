// How the batch's attention work is cut into equal ranges, and how the pieces
// of a shared context are put together again (attn_mfma.hip, attn_stream.hip).
//
// The units are the key steps of every (request, KV head, row chunk), in that
// order, cut into contiguous equal ranges, one per worker (workgroup).  With
// `by_head` the heads are cut alike and worker w * Hkv + g takes range w of head
// g, so that the heads' workgroups walk the same pages side by side: 3 % faster at
// 128 requests x 8 heads of 128 where four waves share a stream, 5 % slower at 256
// requests x 8 heads of 64 with a stream per wave.
// A worker finds its range by a wave scan over the requests: there
// is no plan kernel and no work queue.  A range that covers a part of a chunk's
// steps leaves a partial (m, l, unnormalised o); a worker has at most two (its
// first and its last chunk), so the partials' size depends on the grid and not on
// the contexts.  attn_merge combines them in key order (bitwise reproducible)
// after a kernel boundary, which needs no device-scope fences (on this part those
// write back and invalidate the whole L2 of an XCD).
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace dspark {

constexpr int kRangeCUs = 256;  // gfx950; sizes the grids and the partials
// Batches whose contexts are bounded by this many keys take a worker per (request,
// head, chunk): a worker's few steps cost less than the merge kernel would.
constexpr int kDirectKeys = 256;
// Their grid: (request, head) by chunk, the chunks last, so that what requests leave empty
// of them is the grid's end (next to each other, every second workgroup of 192 requests x
// 8 heads with two chunks was empty and half of the XCDs idle: 72 against 44 us).
constexpr int kDirectChunks = 65535;  // a grid's second dimension, at most
// (request, head) pairs, fewer than: the grids over them are of 256 threads each, and a
// launch takes fewer than 2^32 threads a dimension.
constexpr int64_t kRangePairs = (int64_t)1 << 24;

struct Ranges {
    AttnArgs a;
    int group, chunk_rows;    // query heads per KV head; rows of a chunk
    int by_head;              // every head is cut alike
    int direct;               // short contexts: a worker per (request, head, chunk), no cuts and no merge
    int resident, min_units;  // ranges (per head with by_head), at most; units of a range, at least
    int64_t* head;            // [0] units per range, [32 + r] first unit of request r (written by the workers)
    float* part;              // [worker][2] {m[chunk_rows], l[chunk_rows], o[chunk_rows][Dp]}
};

static inline size_t range_head_bytes(int R) { return (256 + (size_t)R * 8 + 255) & ~(size_t)255; }

__device__ __forceinline__ int range_total_rows(const AttnArgs& a) { return min(max(a.cu_q[a.R], 0), a.R * a.max_q); }

// Shape of request r: false when it is malformed (ql outside [1, max_q], kv
// outside [ql, max_pages * page], rows outside [0, min(cu_q[R], R * max_q))).
__device__ __forceinline__ bool range_shape(const AttnArgs& a, int r, int total_rows, int& q0, int& ql, int& kv) {
    q0 = a.cu_q[r];
    ql = a.cu_q[r + 1] - q0;
    kv = a.kv_len[r];
    if (ql < 1 || ql > a.max_q || kv < ql || kv > a.max_pages * a.page) return false;
    return q0 >= 0 && (int64_t)q0 + ql <= total_rows;
}

template <int STEP>
__device__ __forceinline__ int64_t range_units(const Ranges& p, int r, int total_rows) {
    int q0, ql, kv;
    if (!range_shape(p.a, r, total_rows, q0, ql, kv)) return 0;
    const int ns = (kv + STEP - 1) / STEP;
    const int nrc = (ql * p.group + p.chunk_rows - 1) / p.chunk_rows;
    return (int64_t)(p.by_head ? 1 : p.a.Hkv) * nrc * ns;  // below 2^31 (checked on the host)
}

// Units [u0, u1) of range w, the request r that holds u0 and r's first unit ur;
// false when the range is empty.  Collective over a wave; the values are uniform.
template <int STEP>
__device__ __forceinline__ bool range_find(const Ranges& p, int w, int total_rows, int64_t& u0,
                                           int64_t& u1, int& r, int64_t& ur) {
    const int lane = threadIdx.x & (DSPARK_WAVE - 1);
    const int R = p.a.R;
    const int64_t n0 = lane < R ? range_units<STEP>(p, lane, total_rows) : 0;
    int64_t total = n0;
    for (int b = DSPARK_WAVE; b < R; b += DSPARK_WAVE)
        total += b + lane < R ? range_units<STEP>(p, b + lane, total_rows) : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, DSPARK_WAVE);
    int64_t per = (total + p.resident - 1) / p.resident;
    if (per < p.min_units) per = p.min_units;
    if (blockIdx.x == 0 && threadIdx.x == 0) p.head[0] = per;
    u0 = w * per;
    if (u0 >= total) return false;
    u1 = min(total, u0 + per);
    int64_t before = 0;
    for (int b = 0; b < R; b += DSPARK_WAVE) {
        int64_t n = n0;
        if (b > 0) n = b + lane < R ? range_units<STEP>(p, b + lane, total_rows) : 0;
        int64_t incl = n;
#pragma unroll
        for (int o = 1; o < DSPARK_WAVE; o <<= 1) {
            const int64_t t = __shfl_up(incl, o, DSPARK_WAVE);
            if (lane >= o) incl += t;
        }
        const unsigned long long hit = __ballot(before + incl > u0);
        if (hit) {
            const int l = (int)__builtin_ctzll(hit);
            r = __builtin_amdgcn_readfirstlane(b + l);
            ur = before + __shfl(incl - n, l, DSPARK_WAVE);
            return true;
        }
        before += __shfl(incl, DSPARK_WAVE - 1, DSPARK_WAVE);
    }
    return false;  // not reached: u0 < total
}

// Calls f(r, g, rc, q0, ql, kv, s0, s1, ns, slot) for the parts of chunks in
// this worker's range, in order: steps [s0, s1) of the chunk's ns; the partial,
// when they are not all, goes to `slot` (0: it starts inside the chunk, so it
// is the worker's first; 1: it ends inside, its last).
template <int STEP, typename F>
__device__ __forceinline__ void range_walk(const Ranges& p, F f) {
    const AttnArgs& a = p.a;
    const int total_rows = range_total_rows(a);
    if (p.direct) {
        const int rc = blockIdx.y, g = blockIdx.x % a.Hkv, r = blockIdx.x / a.Hkv;
        int q0, ql, kv;
        if (!range_shape(a, r, total_rows, q0, ql, kv) || rc * p.chunk_rows >= ql * p.group) return;
        const int ns = (kv + STEP - 1) / STEP;
        f(r, g, rc, q0, ql, kv, 0, ns, ns, (int64_t)0);
        return;
    }
    const int heads = p.by_head ? 1 : a.Hkv;  // of this worker's list
    int64_t u0, u1, ur;
    int r;
    if (!range_find<STEP>(p, p.by_head ? blockIdx.x / a.Hkv : blockIdx.x, total_rows, u0, u1, r, ur)) return;
    int64_t u = u0;
    while (u < u1) {  // (r stays below R: the requests from r on hold the units up to u1)
        int q0, ql, kv;
        const bool ok = range_shape(a, r, total_rows, q0, ql, kv);
        const int ns = (kv + STEP - 1) / STEP;
        const int nrc = (ql * p.group + p.chunk_rows - 1) / p.chunk_rows;
        const int units = ok ? heads * nrc * ns : 0;
        if (ok && threadIdx.x == 0) p.head[32 + r] = ur;
        int local = (int)(u - ur);
        while (local < units && u < u1) {
            const int item = local / ns;
            const int s0 = local - item * ns;
            const int gl = item / nrc;
            const int g = p.by_head ? (int)(blockIdx.x % a.Hkv) : gl;
            const int s1 = (int)min((int64_t)ns, s0 + (u1 - u));
            f(r, __builtin_amdgcn_readfirstlane(g), __builtin_amdgcn_readfirstlane(item - gl * nrc), __builtin_amdgcn_readfirstlane(q0),
              __builtin_amdgcn_readfirstlane(ql), __builtin_amdgcn_readfirstlane(kv),
              __builtin_amdgcn_readfirstlane(s0), __builtin_amdgcn_readfirstlane(s1), __builtin_amdgcn_readfirstlane(ns),
              2 * (int64_t)blockIdx.x + (s0 == 0));
            local += s1 - s0;
            u += s1 - s0;
        }
        ur += units;
        ++r;
    }
}

// Combines the partials of every chunk whose steps several ranges share, in
// key order.  Workgroups (request and head, part of the rows); a thread takes
// four values of a row; up to kMergeBatch partials are in flight.  A chain of
// dependent loads, so the rows are spread over up to kMergeParts workgroups.
constexpr int kMergeThreads = 256;
constexpr int kMergeBatch = 8;
constexpr int kMergeParts = 8;
template <bool F32, int ROWS, int DP, int STEP>
__global__ __launch_bounds__(kMergeThreads) void attn_merge(Ranges p) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int64_t kSlot = (int64_t)ROWS * (DP + 2);
    const AttnArgs& a = p.a;
    const int r = blockIdx.x / a.Hkv, g = blockIdx.x % a.Hkv;
    const int64_t per = p.head[0], ur = p.head[32 + r];
    int q0, ql, kv;
    if (!range_shape(a, r, range_total_rows(a), q0, ql, kv)) return;
    const int ns = (kv + STEP - 1) / STEP;
    const int rows = ql * p.group;
    const int nrc = (rows + ROWS - 1) / ROWS;
    const int groups = a.Dv / 4;
    for (int i = blockIdx.y * kMergeThreads + threadIdx.x; i < rows * groups; i += gridDim.y * kMergeThreads) {
        const int row = i / groups, c4 = (i - row * groups) * 4;
        const int rc = row / ROWS, rr = row - rc * ROWS;
        const int64_t c0 = ur + (int64_t)((p.by_head ? 0 : g * nrc) + rc) * ns;  // the chunk's units [c0, c0 + ns)
        const int64_t w0 = c0 / per, w1 = (c0 + ns - 1) / per;
        if (w0 == w1) continue;  // one range had them all: its worker wrote the rows
        float M = -__builtin_huge_valf(), L = 0.0f;
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int64_t w = w0; w <= w1; w += kMergeBatch) {
            float ms[kMergeBatch], ls[kMergeBatch];
            f32x4 os[kMergeBatch];
#pragma unroll
            for (int k = 0; k < kMergeBatch; ++k) {
                const int64_t wk = min(w + k, w1);
                const float* sl = p.part + (2 * (p.by_head ? wk * a.Hkv + g : wk) + (wk == w0)) * kSlot;
                ms[k] = sl[rr];
                ls[k] = sl[ROWS + rr];
                os[k] = *(const f32x4*)(sl + 2 * ROWS + (int64_t)rr * DP + c4);
            }
            float Mb = M;
#pragma unroll
            for (int k = 0; k < kMergeBatch; ++k)
                if (w + k <= w1) Mb = vmax(Mb, ms[k]);
            // rescale what earlier batches accumulated
            if (M > -__builtin_huge_valf() && Mb != M) {
                const float f = exp2f(M - Mb);
                L *= f;
                o *= f;
            }
            M = Mb;
#pragma unroll
            for (int k = 0; k < kMergeBatch; ++k) {
                if (w + k > w1) break;
                const float f = ms[k] == -__builtin_huge_valf() ? 0.0f : exp2f(ms[k] - M);
                L += ls[k] * f;
                o += f * os[k];
            }
        }
        const int t = row / p.group;
        const int64_t orow = (int64_t)(q0 + t) * a.Hq + g * p.group + (row - t * p.group);
        const float inv = 1.0f / L;
        if (F32) *(f32x4*)((float*)a.out + orow * a.Dv + c4) = o * inv;
        else
            *(uint2*)((uint16_t*)a.out + orow * a.Dv + c4) =
                uint2{pack2_bf16(o[0] * inv, o[1] * inv), pack2_bf16(o[2] * inv, o[3] * inv)};
        if (a.lse && c4 == 0) a.lse[orow] = (M + log2f(L)) * 0.6931471805599453f;
    }
}

template <bool F32, int ROWS, int DP, int STEP>
static hipError_t launch_merge(const Ranges& p, hipStream_t s) {
    const int64_t quads = (int64_t)p.a.max_q * p.group * (p.a.Dv / 4);  // of a (request, head), at most
    const int64_t parts = quads / kMergeThreads + (quads % kMergeThreads != 0);
    hipLaunchKernelGGL((attn_merge<F32, ROWS, DP, STEP>),
                       dim3((unsigned)(p.a.R * p.a.Hkv), (unsigned)(parts < kMergeParts ? parts : kMergeParts)),
                       dim3(kMergeThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace dspark
