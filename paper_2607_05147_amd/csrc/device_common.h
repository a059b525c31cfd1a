// Device-side helpers shared by the gfx950 kernels of the verification step.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define DSPARK_WAVE 64

namespace dspark {

// bfloat16 <-> fp32.  Widening is exact; narrowing rounds to nearest even
// (NaN stays NaN).
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(((uint32_t)b) << 16);
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    __device__ __forceinline__ static float load(const float* p, int64_t i) { return p[i]; }
    __device__ __forceinline__ static void store(float* p, int64_t i, float v) { p[i] = v; }
};
template <> struct Elem<uint16_t> {
    __device__ __forceinline__ static float load(const uint16_t* p, int64_t i) {
        return bf16_to_f32(p[i]);
    }
    __device__ __forceinline__ static void store(uint16_t* p, int64_t i, float v) {
        p[i] = f32_to_bf16(v);
    }
};

// Wave-wide reductions over 64 lanes (every lane gets the result).
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, DSPARK_WAVE));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, DSPARK_WAVE);
    return v;
}
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, DSPARK_WAVE);
    return v;
}

// Intra-wave LDS exchange: orders this wave's LDS writes before its later
// LDS reads (DS instructions of one wave execute in order; this stops the
// compiler from moving accesses across the point).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup barrier that orders LDS only: waits for this wave's LDS accesses
// (lgkmcnt) but leaves global loads in flight, so prefetched data keeps
// streaming across the barrier (a plain __syncthreads() waits for every
// outstanding global load as well).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Pointer into LDS (address space 3) from a 32-bit LDS byte address.
template <typename T>
__device__ __forceinline__ T* lds_ptr(uint32_t addr) {
    return (T*)(uintptr_t)addr;
}

// ---- helpers of the matrix-core attention kernels

// 16-byte copy global -> LDS for a whole wave: lane L's 16 bytes land at
// lds_addr + 16 L (lds_addr is wave-uniform).  Emitted as inline asm so that
// the compiler does not add its own conservative waits for it; the kernels
// wait for these copies with explicit vmcnt counts.  The copy reads m0 no sooner than
// one wait state after it is written, and the compiler adds none inside the block.
__device__ __forceinline__ void lds_copy16(const void* gsrc, uint32_t lds_addr) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off"
        :
        : "s"(m0), "v"(gsrc)
        : "memory", "m0");
}

// a wave-uniform 64-bit value, in scalar registers
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// the same with a wave-uniform 64-bit base (SGPRs) and a per-lane 32-bit offset.  The
// base has to come from scalar arithmetic: a vector instruction's write of it would need
// five wait states before the copy, which the compiler does not add inside the block.
__device__ __forceinline__ void lds_copy16_s(uint64_t sbase, uint32_t voff, uint32_t lds_addr) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
    const uint64_t sb = uniform64(sbase);
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2"
        :
        : "s"(m0), "v"(voff), "s"(sb)
        : "memory", "m0");
}

// s_waitcnt vmcnt(N) leaving the other counters alone (gfx9 encoding)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// NaN-propagating maximum (v_maximum3_f32; no operand canonicalisation)
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// max over the four lanes that share a row (lanes lr, lr + 16, lr + 32, lr + 48)
__device__ __forceinline__ float row_max4(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = vmax(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return vmax(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

}  // namespace dspark
