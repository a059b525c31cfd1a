// Ragged causal verify attention on gfx950 matrix cores for any head size up
// to 256 and any page of 16-key blocks, bf16 and fp32: the shapes that the
// head-dim-128 and latent kernels do not take (small heads, 16-token pages,
// unequal key and value sizes, fp32).  Bound by HBM: the packed rows
// (verify tokens x GQA group, row = t * group + head) share one read of the
// request's keys and values.
//
// Work unit = one step (32 keys bf16, 16 keys fp32) of one (request, KV head,
// row chunk of 16 * NT rows); the batch's units are cut into equal ranges, one
// per worker (attn_ranges.h).  A worker is a single wave with its own K and V
// buffers, so nothing in its loop waits for another wave.  Contexts that are
// short for the whole batch (kDirectKeys) take one wave each and no merge.
//
//   * K and V rows are copied from their page straight into LDS
//     (global_load_lds_dwordx4), one step ahead.  A 16-key half step lies
//     inside one page, so a copy needs one uniform page base and per-lane
//     offsets that never change.  Rows are 16 * CH bytes (padded head sizes are
//     filled from a zero block), chunks XOR-swizzled by the copy so that the
//     operand reads are free of bank conflicts.
//   * bf16: S^T = K Q^T and O^T += V^T P^T on v_mfma_f32_16x16x32_bf16.  P enters
//     its product as two bf16 terms, p to within 2^-17 (its sum adds p itself):
//     the output's rounding is 2^-9, and the errors against 64 bits are those of
//     the vector-ALU kernels, whose p is fp32.
//   * fp32: v_mfma_f32_16x16x4_f32 throughout; the score accumulator (keys
//     4 lq + e) is already the B operand of the value product over those keys.
//   * softmax online in exp2 units, the running maximum moved only when it
//     grows by more than 2^8 (exact after the final normalisation);
//   * a worker that finds a sum non-finite computes its rows again key by key
//     (attend_rows), so that a non-finite value reaches only the rows that see it.
//
// Measured (GPU time of the whole call) against the vector-ALU kernels:
//   64 requests, 32/8 heads of 64, 16-key token-major pages, 512-4096 keys, bf16:
//   1690 -> 73-75 us (303 MB, 4.1 TB/s; four times the requests: 4.65 TB/s);
//   16 requests, 32/8 heads of 128, 64-key pages, 512-2048 keys, fp32: 1150 -> 64 us (170 MB, 2.7 TB/s;
//   four times the requests: 4.0 TB/s).
#include <algorithm>
#include <type_traits>

#include "attn_ranges.h"

namespace dspark {
namespace stream {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kRescale = 8.0f;     // log2 headroom before the running max is moved
constexpr int kMinUnits = 4;         // steps per wave, at least
constexpr int kPageRegs = 2;         // page ids per lane: 128 pages in flight of a range
constexpr int kMaxD = 256;

// CH: 16-byte chunks of an LDS row.  bf16: head sizes up to 8 * CH, 32 keys a
// step; fp32: up to 4 * CH, 16 keys a step.
template <bool F32, int CH>
struct Cfg {
    static constexpr int S = CH / 4;            // operand slices of a key row; copy instructions of 16 rows
    static constexpr int H = F32 ? 1 : 2;       // 16-key halves of a step
    static constexpr int Step = 16 * H;
    static constexpr int RowB = 16 * CH;
    static constexpr int TileB = Step * RowB;
    static constexpr int Dp = F32 ? 4 * CH : 8 * CH;  // padded head size
    static constexpr int DB = Dp / 16;
    // single-wave workgroups that a CU's 160 KB of LDS holds
    static constexpr int LdsWaves = 160 * 1024 / (2 * TileB);
    // operand groups: key slices and output blocks read from LDS at a time
    static constexpr int KS = S % 4 == 0 ? 4 : S <= 4 ? S : S / 2, VD = F32 ? 4 : DB % 8 == 0 ? 8 : DB;
    // distinct operand addresses: those that the swizzle's chunk bits reach
    static constexpr int KA = S < 4 || S % 4 ? S : 4, VA = F32 ? 1 : DB % 8 ? DB : 8;
    // registers: accumulators, queries and probabilities of NT row tiles; operands; copy offsets
    static constexpr int regs(int nt) {
        return nt * (4 * DB + 4 * S + 4 * H) + (4 * H * KS > 4 * VD ? 4 * H * KS : 4 * VD) + 2 * H * S;
    }
    // waves per SIMD that the registers allow where LDS does, and waves per CU
    static constexpr int eu(int nt) {
        return regs(nt) <= 90 && LdsWaves > 8 ? 3 : regs(nt) <= 170 && LdsWaves > 5 ? 2 : 1;
    }
    static constexpr int cu(int nt) { return LdsWaves < 4 * eu(nt) ? LdsWaves : 4 * eu(nt); }
};

struct Params : Ranges {
    int64_t ks1b, vs1b;              // KV strides in bytes
    uint32_t ks0b, vs0b, ks2b, vs2b;
    int kbytes, vbytes;              // bytes of a key / value row
    int pad;                         // some row is shorter than the LDS row
    float scale2;
};

// Physical chunk of chunk c in LDS row t: XORs that keep c inside its aligned
// group of 4, 8 or 16 chunks.  gfx950 serves a 16-byte LDS read in four 16-lane
// phases (lanes split by bit 5 and the parity of bits 2 ^ 3 ^ 4) and a
// transposing 8-byte read in two 32-lane halves, over 64 four-byte banks.
// With these, the lanes of every phase of the reads below are on distinct
// banks: a row of 8 (mod 16) chunks leaves the bank half to t's parity, a row
// of 12 chunks spreads four rows by itself, a row of 16 or 32 none.
template <bool F32, int CH>
__device__ __forceinline__ int k_slot(int t, int c) {
    if (F32) return c ^ (t & 15);
    if (CH % 16 == 0) return c ^ ((t & 3) | (((t >> 3) & 3) << 2));
    if (CH % 8 == 0) return c ^ (((t >> 1) & 1) | (((t >> 3) & 3) << 1));
    return c ^ (((t >> 4) & 1) * 3);
}
template <bool F32, int CH>
__device__ __forceinline__ int v_slot(int t, int c) {
    if (F32) return c;
    if (CH % 16 == 0) return c ^ (((t & 3) | (((t >> 3) & 1) << 2)) << 1);
    if (CH % 8 == 0) return c ^ ((((t >> 1) & 1) | (((t >> 3) & 1) << 1)) << 1);
    return c ^ (((t >> 3) & 1) << 1);
}

// 16 bytes of zeros (zero-initialised at load, never written): keys at or past
// the context's end and the pad of short rows are copied from here.
__device__ __align__(16) uint32_t g_zero[4];

// The wait is the builtin, which the compiler counts: with every ordinary load
// waited for before the step loop, it adds no wait of its own inside it.
template <int N>
__device__ __forceinline__ void wait_copies() {
    wait_vmcnt<N>();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The rows of a chunk over the same steps key by key on the vector ALUs, where the
// products above came out non-finite: a product over 16 rows and 32 keys also multiplies
// the keys that a row does not see, by a probability of 0, and 0 times a non-finite value
// is NaN, as is an infinity times the second term of a probability.  Every row takes only
// its own keys here, as the vector-ALU kernels do.
template <bool F32, int CH, int NT>
__device__ __forceinline__ void attend_rows(const Params& p, const int r, const int g, const int rc, const int q0,
                                            const int ql, const int kv, const int s0, const int s1, const int ns,
                                            const int64_t slot) {
    typedef Cfg<F32, CH> C;
    typedef typename std::conditional<F32, float, uint16_t>::type T;
    constexpr int kPer = (C::Dp + DSPARK_WAVE - 1) / DSPARK_WAVE;  // value dims per lane
    const AttnArgs& a = p.a;
    // (values in vector registers: the scalar ones that this would add to the kernel's
    // are spilled into vector registers that the step loop then lacks)
    int z = 0;
    asm volatile("" : "+v"(z));
    const int lane = threadIdx.x, page = a.page + z, group = p.group + z, gv = g + z;
    const int row0 = (rc + z) * (16 * NT), nrows = min(16 * NT, ql * group - row0);
    const int32_t* bt = a.block_table + (int64_t)(r + z) * a.max_pages;
    const T* kc = (const T*)a.k + gv * a.ks[1];
    const T* vc = (const T*)a.v + gv * a.vs[1];
    const bool whole = s0 + z == 0 && s1 == ns;
    float* part = p.part + (slot + z) * ((int64_t)(16 * NT) * (C::Dp + 2));
    for (int rr = 0; rr < nrows; ++rr) {
        const int row = row0 + rr, t = row / group;
        const int64_t orow = (int64_t)(q0 + t) * a.Hq + gv * group + (row - t * group);
        const int end = min(kv - ql + t + 1, s1 * C::Step);
        float m = -__builtin_huge_valf(), l = 0.0f, o[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) o[e] = 0.0f;
        for (int k0 = (s0 + z) * C::Step; k0 < end; k0 += DSPARK_WAVE) {
            const int key = min(k0 + lane, end - 1);
            const T* kr = kc + (int64_t)bt[key / page] * a.ks[0] + (int64_t)(key % page) * a.ks[2];
            float sc = 0.0f;
            for (int d = 0; d < a.Dqk + z; ++d)
                sc += Elem<T>::load((const T*)a.q, orow * a.Dqk + d) * p.scale2 * Elem<T>::load(kr, d);
            if (k0 + lane >= end) sc = -__builtin_huge_valf();
            const float mn = fmaxf(m, wave_max(sc));
            const float alpha = m == -__builtin_huge_valf() ? 0.0f : exp2f(m - mn);
            const float pr = sc == -__builtin_huge_valf() ? 0.0f : exp2f(sc - (mn == -__builtin_huge_valf() ? 0.0f : mn));
            l = l * alpha + wave_sum(pr);
            m = mn;
#pragma unroll
            for (int e = 0; e < kPer; ++e) o[e] *= alpha;
            for (int j = 0; j < min(DSPARK_WAVE, end - k0); ++j) {
                const T* vr = vc + (int64_t)bt[(k0 + j) / page] * a.vs[0] + (int64_t)((k0 + j) % page) * a.vs[2];
                const float pj = __shfl(pr, j, DSPARK_WAVE);
#pragma unroll
                for (int e = 0; e < kPer; ++e) {
                    const int d = lane + e * DSPARK_WAVE;
                    if (d < a.Dv) o[e] += pj * Elem<T>::load(vr, d);
                }
            }
        }
        if (lane == 0) {
            if (!whole) part[rr] = m, part[16 * NT + rr] = l;
            else if (a.lse) a.lse[orow] = (m + log2f(l)) * kLn2;
        }
        const float inv = 1.0f / l;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int d = lane + e * DSPARK_WAVE;
            if (d >= a.Dv) continue;
            if (whole) Elem<T>::store((T*)a.out, orow * a.Dv + d, o[e] * inv);
            else part[2 * 16 * NT + rr * C::Dp + d] = o[e];
        }
    }
}

// Steps [s0, s1) of the ns steps of one (request, head, chunk).  `slot`: where
// the partial goes when they are not all of them.  Returns whether a sum of its rows is
// not finite (what is written is then not yet the result).
template <bool F32, int CH, int NT>
__device__ __forceinline__ bool attend(const Params& p, const uint32_t lds0, const int r, const int g, const int rc,
                                       const int q0, const int ql, const int kv, const int s0, const int s1,
                                       const int ns, const int64_t slot) {
    typedef Cfg<F32, CH> C;
    constexpr int S = C::S, H = C::H;
    const AttnArgs& a = p.a;
    const int lane = threadIdx.x;
    const int lr = lane & 15, lq = lane >> 4;
    const int rows = ql * p.group;
    const int row0 = rc * (16 * NT);
    const int nt = min(NT, (rows - row0 + 15) >> 4);

    // ---- query fragments (B operand of S^T = K Q^T) and causal limits
    // bf16: dims 32 s + 8 lq ..; fp32: dims 16 s + 4 lq ..
    u32x4 qf[NT][S];
    int lim[NT];
    int lim_min = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int row = row0 + 16 * j + lr;
        lim[j] = -1;
#pragma unroll
        for (int s = 0; s < S; ++s) qf[j][s] = u32x4{0u, 0u, 0u, 0u};
        if (row < rows) {
            const int t = row / p.group;
            const int h = g * p.group + (row - t * p.group);
            const char* qp = (const char*)a.q + ((int64_t)(q0 + t) * a.Hq + h) * p.kbytes + 16 * lq;
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (64 * s + 16 * lq < p.kbytes) qf[j][s] = *(const u32x4*)(qp + 64 * s);
            lim[j] = kv - ql + t;
            lim_min = min(lim_min, lim[j]);
        }
    }
    lim_min = __reduce_min_sync(~0ull, lim_min);
    // with one wave per SIMD the queries live in the accumulation registers
    // (the products read them from there)
    if constexpr (C::eu(NT) == 1) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int s = 0; s < S; ++s) asm volatile("" : "+a"(qf[j][s]));
    }

    f32x4 acc[NT][C::DB];
    float mrow[NT], lsum[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        mrow[j] = -__builtin_huge_valf();
        lsum[j] = 0.0f;
#pragma unroll
        for (int d = 0; d < C::DB; ++d) acc[j][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // ---- copy offsets from a half step's first key: instruction i covers chunks
    // 64 i + lane of the half's 16 rows
    uint32_t ko[H][S], vo[H][S];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int t = (64 * i + lane) / CH, c = (64 * i + lane) % CH;
            ko[h][i] = t * p.ks2b + 16 * k_slot<F32, CH>(t + 16 * h, c);  // the maps are involutions
            vo[h][i] = t * p.vs2b + 16 * v_slot<F32, CH>(t + 16 * h, c);
        }
    // LDS addresses of the operand reads: the swizzles leave bit 2 of the key (the
    // key block, the half of a transposing read) and the high chunk bits alone,
    // so those are immediate offsets
    uint32_t kaddr[C::KA], vaddr[C::VA];
#pragma unroll
    for (int i = 0; i < C::KA; ++i) {
        const int t = F32 ? lr : 8 * (lr >> 2) + (lr & 3);
        kaddr[i] = lds0 + t * C::RowB + 16 * k_slot<F32, CH>(t, 4 * i + lq);
    }
#pragma unroll
    for (int i = 0; i < C::VA; ++i) {
        const int t = F32 ? 4 * lq : 8 * lq + (lr >> 2), c = F32 ? lr : 2 * i + ((lr & 3) >> 1);
        vaddr[i] = lds0 + C::TileB + t * C::RowB + 16 * v_slot<F32, CH>(t, c) + (F32 ? 0 : 8 * (lr & 1));
    }
    const uint64_t k_head = (uint64_t)(uintptr_t)a.k + (uint64_t)(g * p.ks1b);
    const uint64_t v_head = (uint64_t)(uintptr_t)a.v + (uint64_t)(g * p.vs1b);

    for (int sb = s0; sb < s1;) {
        // the page ids of up to 128 pages from the segment's first, two per lane
        const int pg0 = sb * C::Step / a.page;
        const int pg_last = (kv - 1) / a.page;
        const int64_t seg_end = (int64_t)(pg0 + kPageRegs * DSPARK_WAVE) * a.page / C::Step;
        const int se = (int)min((int64_t)s1, seg_end);
        int pgs[kPageRegs];
#pragma unroll
        for (int k = 0; k < kPageRegs; ++k) {
            const int pg = pg0 + k * DSPARK_WAVE + lane;
            pgs[k] = pg <= pg_last ? a.block_table[(int64_t)r * a.max_pages + pg] : 0;
        }
        const int nseg = se - sb;
        // the half steps to issue next: first key, page (relative) and slot
        int ikey = sb * C::Step;
        int ipg = 0, islot = ikey - pg0 * a.page;
        uint64_t kslot = (uint64_t)islot * p.ks2b, vslot = (uint64_t)islot * p.vs2b;  // bytes
        uint64_t vbase[H];
        int vkey = 0;
        auto copy = [&](uint64_t base, uint32_t (&off)[H][S], int h, int key0, uint32_t dst, auto slot, int bytes) {
            if (key0 + 16 <= kv && !p.pad) {
#pragma unroll
                for (int i = 0; i < S; ++i) lds_copy16_s(base, off[h][i], dst + (h * S + i) * 1024);
            } else {
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    const int t = (64 * i + lane) / CH, c = (64 * i + lane) % CH;
                    const bool in = key0 + t < kv && 16 * slot(t + 16 * h, c) < bytes;
                    lds_copy16(in ? (const void*)(uintptr_t)(base + off[h][i]) : (const void*)g_zero,
                               dst + (h * S + i) * 1024);
                }
            }
        };
        auto issue_k = [&]() {
            vkey = ikey;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int lo = __builtin_amdgcn_readlane(pgs[0], ipg & 63);
                const int hi = __builtin_amdgcn_readlane(pgs[1], ipg & 63);
                const uint32_t page = ipg < DSPARK_WAVE ? lo : hi;
                vbase[h] = v_head + (uint64_t)page * p.vs0b + vslot;
                copy(k_head + (uint64_t)page * p.ks0b + kslot, ko, h, ikey, lds0, k_slot<F32, CH>, p.kbytes);
                ikey += 16;
                islot += 16;
                kslot += 16 * p.ks2b;  // 16 keys: below 2^32 bytes
                vslot += 16 * p.vs2b;
                if (islot >= a.page) {
                    islot = 0;
                    kslot = vslot = 0;
                    ++ipg;
                }
            }
        };
        auto issue_v = [&]() {
#pragma unroll
            for (int h = 0; h < H; ++h)
                copy(vbase[h], vo, h, vkey + 16 * h, lds0 + C::TileB, v_slot<F32, CH>, p.vbytes);
        };

        // ---- the segment.  One K and one V buffer: a buffer is refilled for the
        // next step as soon as this step's operands are in registers, so the next
        // K lands during the softmax and the value product and the next V during
        // the next scores.  Copies land in order: with V (or the next K) issued
        // after it, K (or V) has landed at vmcnt <= the copies of one tile.
        wait_copies<0>();
        issue_k();
        issue_v();
        for (int n = 0; n < nseg; ++n) {
            const int tok0 = (sb + n) * C::Step;
            const bool more = n + 1 < nseg;
            const bool full = tok0 + C::Step <= kv && tok0 + C::Step - 1 <= lim_min;
            constexpr int kNS = F32 ? 4 : 8;  // scores per lane and tile
            u32x4 pb[NT][H];              // probabilities, operands of the value product
            wait_copies<H * S>();  // K of step n
            // scores of tile j: bf16 keys tok0 + 8 lq + x (two key blocks), fp32 keys
            // tok0 + 4 lq + x (even and odd slices) of query row lr
            auto dot = [&](int j, f32x4 (&sc)[2], u32x4 (&kf)[H][C::KS], int s0) {
#pragma unroll
                for (int s = 0; s < C::KS; ++s) {
                    if constexpr (F32) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                __uint_as_float(kf[0][s][e]), __uint_as_float(qf[j][s0 + s][e]), sc[s & 1], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int mb = 0; mb < H; ++mb)
                            sc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[mb][s]),
                                                                           __builtin_bit_cast(bf16x8, qf[j][s0 + s]),
                                                                           sc[mb], 0, 0, 0);
                    }
                }
            };
            auto softmax = [&](int j, f32x4 (&sc)[2]) {
                if constexpr (F32) sc[0] += sc[1];
                float sv[kNS];
#pragma unroll
                for (int x = 0; x < kNS; ++x) sv[x] = sc[x >> 2][x & 3];
                if (!full) {
#pragma unroll
                    for (int x = 0; x < kNS; ++x) {
                        const int key = tok0 + kNS * lq + x;
                        if (!(key < kv && key <= lim[j])) sv[x] = -__builtin_huge_valf();
                    }
                }
                float bm = vmax(vmax(sv[0], sv[1]), vmax(sv[2], sv[3]));
                if constexpr (!F32) bm = vmax(bm, vmax(vmax(sv[4], sv[5]), vmax(sv[6], sv[7])));
                bm = row_max4(bm) * p.scale2;
                const bool need = bm > mrow[j] + kRescale;
                if (__builtin_amdgcn_ballot_w64(need)) {
                    const float mn = need ? bm : mrow[j];
                    const float alpha = need ? __builtin_amdgcn_exp2f(mrow[j] - mn) : 1.0f;
                    lsum[j] *= alpha;
#pragma unroll
                    for (int d = 0; d < C::DB; ++d) acc[j][d] *= alpha;
                    mrow[j] = mn;
                }
                const float mu = mrow[j] == -__builtin_huge_valf() ? 0.0f : mrow[j];
                float pr[kNS];
#pragma unroll
                for (int x = 0; x < kNS; ++x) pr[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[x], p.scale2, -mu));
                lsum[j] += (pr[0] + pr[1]) + (pr[2] + pr[3]);
                if constexpr (!F32) lsum[j] += (pr[4] + pr[5]) + (pr[6] + pr[7]);
                // fp32: p itself; bf16: p = hi + lo
                if constexpr (F32) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) pb[j][0][x] = __float_as_uint(pr[x]);
                } else {
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t hi = cvt_pk_bf16(pr[2 * x], pr[2 * x + 1]);
                        pb[j][0][x] = hi;
                        pb[j][1][x] = cvt_pk_bf16(pr[2 * x] - __uint_as_float(hi << 16),
                                                  pr[2 * x + 1] - __uint_as_float(hi & 0xffff0000u));
                    }
                }
            };
            // K operands of slices s0 ..: bf16 keys 8 (lr / 4) + 4 mb + lr % 4, fp32 key
            // lr; the last ones free the buffer
            auto load_k = [&](u32x4 (&kf)[H][C::KS], int s0) {
#pragma unroll
                for (int mb = 0; mb < H; ++mb)
#pragma unroll
                    for (int s = 0; s < C::KS; ++s)
                        kf[mb][s] = *lds_ptr<const lds_u32x4>(kaddr[(s0 + s) % C::KA] + 4 * mb * C::RowB +
                                                              64 * (s0 + s - (s0 + s) % C::KA));
                if (s0 + C::KS >= S) {
                    wait_lds();
                    if (more) issue_k();
                }
            };
            if constexpr (C::KS == S) {
                u32x4 kf[H][C::KS];
                load_k(kf, 0);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    if (j > 0 && j >= nt) continue;
                    f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                    dot(j, sc, kf, 0);
                    softmax(j, sc);
                }
            } else {  // in groups of slices, which bounds the registers
                f32x4 sc[NT][2];
#pragma unroll
                for (int j = 0; j < NT; ++j) sc[j][0] = sc[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s0 = 0; s0 < S; s0 += C::KS) {
                    u32x4 kf[H][C::KS];
                    load_k(kf, s0);
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        if (j == 0 || j < nt) dot(j, sc[j], kf, s0);
                }
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    if (j == 0 || j < nt) softmax(j, sc[j]);
            }
            if (more) wait_copies<H * S>();  // V of step n
            else wait_copies<0>();
            // the value operands, in groups of output blocks
#pragma unroll
            for (int d0 = 0; d0 < C::DB; d0 += C::VD) {
                u32x4 vf[C::VD];
                if constexpr (!F32) {
                    // transposing reads: dims 16 d + lr, keys 8 lq ..
#pragma unroll
                    for (int d = 0; d < C::VD; ++d) {
                        uint2 hh[2];
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            hh[x] = __builtin_bit_cast(
                                uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<lds_s16x4>(
                                           vaddr[(d0 + d) % C::VA] + 4 * x * C::RowB + 32 * (d0 + d - (d0 + d) % C::VA))));
                        vf[d] = u32x4{hh[0].x, hh[0].y, hh[1].x, hh[1].y};
                    }
                } else {
                    // key 4 lq + e in vf[e]: O^T over those keys, operand row m of block
                    // 4 b + x is dim 64 b + 4 m + x
#pragma unroll
                    for (int e = 0; e < 4; ++e) vf[e] = *lds_ptr<const lds_u32x4>(vaddr[0] + e * C::RowB + 64 * d0);
                }
                if (d0 + C::VD >= C::DB) {
                    wait_lds();
                    if (more) issue_v();
                }
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    if (j > 0 && j >= nt) continue;
                    if constexpr (F32) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int x = 0; x < 4; ++x)
                                acc[j][d0 + x] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(vf[e][x]), __uint_as_float(pb[j][0][e]),
                                                                                    acc[j][d0 + x], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int d = 0; d < C::VD; ++d) {
                            const bf16x8 v = __builtin_bit_cast(bf16x8, vf[d]);
                            acc[j][d0 + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                v, __builtin_bit_cast(bf16x8, pb[j][0]), acc[j][d0 + d], 0, 0, 0);
                            acc[j][d0 + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                v, __builtin_bit_cast(bf16x8, pb[j][H - 1]), acc[j][d0 + d], 0, 0, 0);
                        }
                    }
                }
            }
        }
        sb = se;
    }

    // ---- rows: total l over the four lanes of a row
    const bool whole = s0 == 0 && s1 == ns;
    float* part = p.part + slot * ((int64_t)(16 * NT) * (C::Dp + 2));
    // largest sum by magnitude (NaN if one is), two values an instruction and in independent
    // chains (one chain of a value each cost 0.2 - 0.4 us more a call)
    float big[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        lsum[j] += __shfl_xor(lsum[j], 16, 64);
        lsum[j] += __shfl_xor(lsum[j], 32, 64);
        const int rr = 16 * j + lr, row = row0 + rr;
        if (row >= rows) continue;
        big[0] = vmax(big[0], lsum[j]);
#pragma unroll
        for (int d = 0; d < C::DB; ++d) {
            big[d & 3] = vmax(vmax(__builtin_fabsf(acc[j][d][0]), __builtin_fabsf(acc[j][d][1])), big[d & 3]);
            big[d & 3] = vmax(vmax(__builtin_fabsf(acc[j][d][2]), __builtin_fabsf(acc[j][d][3])), big[d & 3]);
        }
        const int t = row / p.group;
        const int64_t orow = (int64_t)(q0 + t) * a.Hq + g * p.group + (row - t * p.group);
        const float inv = 1.0f / lsum[j];
        if (whole) {
            if (a.lse && lq == 0) a.lse[orow] = (mrow[j] + log2f(lsum[j])) * kLn2;
        } else if (lq == 0) {
            part[rr] = mrow[j];
            part[16 * NT + rr] = lsum[j];
        }
#pragma unroll
        for (int d = 0; d < C::DB; ++d) {
            // four consecutive dims of this lane
            f32x4 o;
            int dim;
            if (F32) {
                dim = 64 * (d >> 2) + 16 * lq + 4 * (d & 3);
#pragma unroll
                for (int x = 0; x < 4; ++x) o[x] = acc[j][(d & ~3) + x][d & 3];
            } else {
                dim = 16 * d + 4 * lq;
                o = acc[j][d];
            }
            if (!whole) {
                *(f32x4*)(part + 2 * 16 * NT + (int64_t)rr * C::Dp + dim) = o;
            } else if (dim < a.Dv) {
                if (F32) *(f32x4*)((float*)a.out + orow * a.Dv + dim) = o * inv;
                else
                    *(uint2*)((uint16_t*)a.out + orow * a.Dv + dim) =
                        uint2{pack2_bf16(o[0] * inv, o[1] * inv), pack2_bf16(o[2] * inv, o[3] * inv)};
            }
        }
    }
    return __builtin_amdgcn_ballot_w64(!(vmax(vmax(big[0], big[1]), vmax(big[2], big[3])) < __builtin_huge_valf())) != 0;
}

template <bool F32, int CH, int NT>
__global__ __launch_bounds__(DSPARK_WAVE) __attribute__((amdgpu_waves_per_eu(Cfg<F32, CH>::eu(NT))))
void attn_stream_kernel(Params p) {
    typedef Cfg<F32, CH> C;
    __shared__ __align__(16) unsigned char lds[2 * C::TileB];
    uint32_t lds0 = (uint32_t)(uintptr_t)&lds[0];
    asm volatile("" : "+s"(lds0));
    bool again = false;
    range_walk<C::Step>(p, [&](int r, int g, int rc, int q0, int ql, int kv, int s0, int s1, int ns, int64_t slot) {
        again |= attend<F32, CH, NT>(p, lds0, r, g, rc, q0, ql, kv, s0, s1, ns, slot);
    });
    if (!again) return;
    // (a walk of its own, so that the step loop above holds none of its registers)
    __syncthreads();  // what the lanes of the wave wrote above comes before what others write below
    range_walk<C::Step>(p, [&](int r, int g, int rc, int q0, int ql, int kv, int s0, int s1, int ns, int64_t slot) {
        attend_rows<F32, CH, NT>(p, r, g, rc, q0, ql, kv, s0, s1, ns, slot);
    });
}

// ------------------------------------------------------------------ host

struct Geom {
    int ch, nt, rc_max, direct;
    int64_t resident, waves;  // ranges; grid of the attention kernel
    size_t part_bytes;
};

// LDS row of the head size: the smallest that holds both the key and the value
static int chunks_of(const AttnArgs& a) {
    const int d = std::max(a.Dqk, a.Dv);
    if (!a.bf16) return d <= 64 ? 16 : d <= 128 ? 32 : 64;
    return d <= 64 ? 8 : d <= 96 ? 12 : d <= 128 ? 16 : d <= 192 ? 24 : 32;
}

template <typename F>
static auto with_cfg(bool bf16, int ch, int nt, F f) {
#define DS_NT(F32, CH, MAX)                                                          \
    do {                                                                             \
        if (nt == 1 || MAX == 1) return f(std::integral_constant<bool, F32>{}, std::integral_constant<int, CH>{}, std::integral_constant<int, 1>{}); \
        if (nt == 2 || MAX == 2) return f(std::integral_constant<bool, F32>{}, std::integral_constant<int, CH>{}, std::integral_constant<int, MAX == 1 ? 1 : 2>{}); \
        return f(std::integral_constant<bool, F32>{}, std::integral_constant<int, CH>{}, std::integral_constant<int, MAX>{}); \
    } while (0)
    if (bf16) {
        if (ch == 8) DS_NT(false, 8, 4);
        if (ch == 12) DS_NT(false, 12, 4);
        if (ch == 16) DS_NT(false, 16, 2);
        if (ch == 24) DS_NT(false, 24, 2);
        DS_NT(false, 32, 1);
    }
    if (ch == 16) DS_NT(true, 16, 4);
    if (ch == 32) DS_NT(true, 32, 2);
    DS_NT(true, 64, 1);
#undef DS_NT
}

static Geom geom(const AttnArgs& a) {
    Geom g;
    g.ch = chunks_of(a);
    const int64_t rows = (int64_t)a.max_q * (a.Hq / a.Hkv);
    const int64_t max_kv = (int64_t)a.max_pages * a.page;
    g.direct = max_kv <= kDirectKeys && (rows + 15) / 16 <= kDirectChunks;
    // row tiles per wave: as many as a request can fill, up to what the
    // registers hold (fp32 heads of 65-128 spill 16 with two tiles; more tiles than
    // these read the keys again, from the last-level cache).  Short contexts have few
    // waves and are bound by a wave's own chain of steps, so each takes one tile.
    const int most = a.bf16 ? (g.ch <= 12 ? 4 : g.ch <= 24 ? 2 : 1) : (g.ch <= 16 ? 4 : g.ch <= 32 ? 2 : 1);
    g.nt = g.direct ? 1 : (int)std::min<int64_t>(rows <= 16 ? 1 : rows <= 32 ? 2 : 4, most);
    g.rc_max = (int)((rows + 16 * g.nt - 1) / (16 * g.nt));
    const int64_t items = (int64_t)a.R * a.Hkv * g.rc_max;
    g.part_bytes = 0;
    with_cfg(a.bf16, g.ch, g.nt, [&](auto f32, auto ch, auto nt) {
        typedef Cfg<decltype(f32)::value, decltype(ch)::value> C;
        const int64_t units = items * ((max_kv + C::Step - 1) / C::Step);
        g.resident = kRangeCUs * C::cu(decltype(nt)::value);
        g.waves = g.direct ? items : std::min<int64_t>(g.resident, (units + kMinUnits - 1) / kMinUnits);
        if (!g.direct) g.part_bytes = (size_t)g.waves * 2 * (16 * decltype(nt)::value) * (C::Dp + 2) * sizeof(float);
        return 0;
    });
    return g;
}

}  // namespace stream

bool attn_stream_shape_ok(const AttnArgs& a) {
    if (std::max(a.Dqk, a.Dv) > stream::kMaxD) return false;
    const stream::Geom g = stream::geom(a);
    // a request's units and the grid fit 32 bits
    return (int64_t)a.Hkv * g.rc_max * (((int64_t)a.max_pages * a.page + 15) / 16) < (int64_t)1 << 31 &&
           g.waves < (int64_t)1 << 31 && (int64_t)a.R * a.Hkv < kRangePairs;
}

bool attn_stream_supported(const AttnArgs& a) {
    if (!attn_stream_shape_ok(a)) return false;
    const int per = a.bf16 ? 8 : 4;  // elements of a 16-byte copy
    for (int i = 0; i < 3; ++i)
        if (a.ks[i] % per || a.vs[i] % per) return false;
    // 32-bit page strides, and offsets inside a 16-key block, in bytes
    const int64_t lim0 = (int64_t)1 << 30, lim2 = (int64_t)1 << 24;
    if (a.ks[0] >= lim0 || a.vs[0] >= lim0 || a.ks[2] >= lim2 || a.vs[2] >= lim2) return false;
    return (uintptr_t)a.q % 16 == 0 && (uintptr_t)a.k % 16 == 0 && (uintptr_t)a.v % 16 == 0 &&
           (uintptr_t)a.out % (a.bf16 ? 8 : 16) == 0;
}

size_t attn_stream_workspace(const AttnArgs& a) {
    const stream::Geom g = stream::geom(a);
    return g.direct ? 0 : range_head_bytes(a.R) + g.part_bytes;
}

hipError_t launch_attn_stream(const AttnArgs& a, void* ws, hipStream_t s) {
    const stream::Geom g = stream::geom(a);
    stream::Params p;
    const int64_t esz = a.bf16 ? 2 : 4;
    p.a = a;
    p.group = a.Hq / a.Hkv;
    p.chunk_rows = 16 * g.nt;
    p.by_head = 0;
    p.resident = (int)g.resident;
    p.min_units = stream::kMinUnits;
    p.direct = g.direct;
    p.ks0b = (uint32_t)(a.ks[0] * esz);
    p.ks1b = a.ks[1] * esz;
    p.vs0b = (uint32_t)(a.vs[0] * esz);
    p.vs1b = a.vs[1] * esz;
    p.ks2b = (uint32_t)(a.ks[2] * esz);
    p.vs2b = (uint32_t)(a.vs[2] * esz);
    p.kbytes = (int)(a.Dqk * esz);
    p.vbytes = (int)(a.Dv * esz);
    p.pad = p.kbytes != 16 * g.ch || p.vbytes != 16 * g.ch;
    p.scale2 = a.scale * stream::kLog2e;
    p.head = (int64_t*)ws;
    p.part = (float*)((char*)ws + range_head_bytes(a.R));
    return stream::with_cfg(a.bf16, g.ch, g.nt, [&](auto f32, auto ch, auto nt) {
        constexpr bool F = decltype(f32)::value;
        constexpr int CH = decltype(ch)::value, NT = decltype(nt)::value;
        const dim3 grid = g.direct ? dim3((unsigned)(a.R * a.Hkv), (unsigned)g.rc_max) : dim3((unsigned)g.waves);
        hipLaunchKernelGGL((stream::attn_stream_kernel<F, CH, NT>), grid, dim3(DSPARK_WAVE), 0, s, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || g.direct) return e;
        return launch_merge<F, 16 * NT, stream::Cfg<F, CH>::Dp, stream::Cfg<F, CH>::Step>(p, s);
    });
}

}  // namespace dspark
