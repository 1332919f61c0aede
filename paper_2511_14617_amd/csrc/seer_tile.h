// Helpers shared by the tiled (matrix-core) verify-attention kernels: operand types, the
// hand-placed synchronisation primitives of the direct-to-LDS tile ring, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "seer_device.h"

namespace seer {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

#define SEER_AS1 __attribute__((address_space(1)))
#define SEER_AS3 __attribute__((address_space(3)))

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    f32x2 v = {lo, hi};
    bf16x2 r = __builtin_convertvector(v, bf16x2);   // round-to-nearest-even (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint32_t, r);
}

// acc + lo + hi of a packed pair of bf16 values, in fp32 (v_dot2_f32_bf16 against the pair (1, 1)): the sum of
// the probabilities exactly as the P.V matrix product will see them, in one instruction per pair.
__device__ __forceinline__ float add_bf16_pair(uint32_t pair, float acc) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, 0x3f803f80u), acc, false);
}

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4 and lgkmcnt 11:8 left at "do not wait").
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Workgroup barrier WITHOUT the memory fences of __syncthreads(): a fence (even one scoped to
// LDS) makes the compiler drain every outstanding load, including the direct-to-LDS loads of
// the tiles still in flight, which is exactly what the ring of stages exists to avoid.  The
// kernel orders its LDS traffic by hand instead: wait_vmcnt for the tile about to be read, then
// this barrier; LDS reads of a stage are complete (their results consumed by MFMAs) before the
// wave reaches the barrier after which that stage is overwritten.
__device__ __forceinline__ void bare_barrier() { __builtin_amdgcn_s_barrier(); }
// A workgroup-uniform 32-bit value read from global memory, moved to a scalar register.  The
// hand-placed fences keep the compiler from proving such loads invariant, so it issues them as
// vector loads; without this the control flow that depends on them would be treated as divergent.
__device__ __forceinline__ int uniform_load(const int32_t* p) { return __builtin_amdgcn_readfirstlane(*p); }

// max over the two lanes that share a query row (lane and lane ^ 32), without touching LDS:
// v_permlane32_swap exchanges the upper 32 lanes of its first operand with the lower 32 lanes of
// its second, so from two copies of x one register ends up with the lower half's values in both
// halves and the other with the upper half's.  (Issued from an asm block: with the builtin this
// compiler keeps only the first of the two results.  The s_nop covers the wait states the
// instruction needs after a vector-ALU write of its operands.)
__device__ __forceinline__ float max_across_halves(float x) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));   // (fmaxf would first quieten both operands: two more instructions)
    return m;
}

// Softmax bookkeeping of one tile for this lane's row, from the row's raw score maximum mx_raw
// (masked slots excluded): moves the exponent reference m_run only when the new maximum exceeds
// it by more than 8 (probabilities then stay below 2^8), returns the reference to subtract (in
// units of log2 e, scores scaled) and leaves in alpha the factor that brings sums taken under the
// old reference to the new one.  scale_log2 > 0.
__device__ __forceinline__ float move_reference(float mx_raw, float scale_log2, float& m_run, float& alpha) {
    const float mx = max_across_halves(mx_raw) * scale_log2;
    const float m_new = (mx > m_run + 8.f) ? mx : m_run;      // m_run = -inf: any finite mx moves it
    const float m_use = (m_new == kNegInf) ? 0.f : m_new;      // nothing visible yet: keep exp2 finite
    alpha = fast_exp2(m_run - m_use);
    m_run = m_new;
    return m_use;
}

}  // namespace seer
