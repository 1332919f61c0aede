// Helpers shared by the tiled (matrix-core) verify-attention kernels: operand types, the
// hand-placed synchronisation primitives of the direct-to-LDS tile ring, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

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

// ---------------------------------------------------------------------------
// Tiles of 32 tokens in LDS, K rows then V rows, for separate K and V pools of any supported head size.
// ---------------------------------------------------------------------------
namespace tile {

constexpr int kTile = 32;

template <int DQK, int DV>
struct Shape {
    static constexpr int kKRow = DQK * 2, kVRow = DV * 2;                    // bytes of a token's row
    static constexpr int kKBytes = kTile * kKRow, kVBytes = kTile * kVRow;
    static constexpr int kStage = kKBytes + kVBytes;
    static constexpr int kKSteps = DQK / 16, kDTiles = DV / 32;
    static_assert(kKRow % 128 == 0 && kVRow % 128 == 0 && kKBytes % 1024 == 0 && kVBytes % 1024 == 0, "");
};

// LDS swizzles: 16-byte chunk c of row r is stored at chunk position c ^ f(r) of the row.  64 banks of 4 bytes are 16
// chunks.  K (ds_read_b128, 16 rows at one chunk per quarter-wave): rows of 256 or 512 bytes all start at bank 0 and take
// four bits of the row; rows of 128 or 384 bytes alternate between two halves of the banks and take three.
// V (transposing read, 4 rows x 64 bytes per half-wave): the four rows must fall into different 64-byte groups.
template <int ROW_BYTES>
__device__ __forceinline__ int k_swz(int row) { return ROW_BYTES % 256 == 0 ? row & 15 : (row >> 1) & 7; }
template <int ROW_BYTES>
__device__ __forceinline__ int v_swz(int row) { return ROW_BYTES % 256 == 0 ? (row & 3) << 2 : ((row >> 1) & 1) << 2; }

__device__ __forceinline__ int lds_addr(const unsigned char* p) {
    return static_cast<int>(reinterpret_cast<uintptr_t>((const SEER_AS3 void*)(p)));
}

// Operand reads and their wait in one block (through the builtins the compiler would put a vmcnt(0) in front of them: it
// cannot tell them apart from the tile loads in flight).
__device__ __forceinline__ void read_k4(u32x4 (&kv)[4], int a0, int a1, int a2, int a3) {
    asm volatile("ds_read_b128 %0, %4\n"
                 "ds_read_b128 %1, %5\n"
                 "ds_read_b128 %2, %6\n"
                 "ds_read_b128 %3, %7\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(kv[0]), "=&v"(kv[1]), "=&v"(kv[2]), "=&v"(kv[3])
                 : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
                 : "memory");
}
// V^T operands of two d-tiles (lane addresses a0, a1) for the tile's 32 tokens: vr[tile][token rows 0, 8, 16, 24].
template <int OFF, int ROW8>
__device__ __forceinline__ void read_v2(u32x2 (&vr)[2][4], int a0, int a1) {
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%10\n"
                 "ds_read_b64_tr_b16 %1, %8 offset:%11\n"
                 "ds_read_b64_tr_b16 %2, %8 offset:%12\n"
                 "ds_read_b64_tr_b16 %3, %8 offset:%13\n"
                 "ds_read_b64_tr_b16 %4, %9 offset:%10\n"
                 "ds_read_b64_tr_b16 %5, %9 offset:%11\n"
                 "ds_read_b64_tr_b16 %6, %9 offset:%12\n"
                 "ds_read_b64_tr_b16 %7, %9 offset:%13\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(vr[0][0]), "=&v"(vr[0][1]), "=&v"(vr[0][2]), "=&v"(vr[0][3]), "=&v"(vr[1][0]),
                   "=&v"(vr[1][1]), "=&v"(vr[1][2]), "=&v"(vr[1][3])
                 : "v"(a0), "v"(a1), "n"(OFF), "n"(OFF + ROW8), "n"(OFF + 2 * ROW8), "n"(OFF + 3 * ROW8)
                 : "memory");
}

// Where a lane finds its operands in a tile: K chunk 2 kk + lg of row ln (step kk: ^ (kk % kPerXor) << 5, + whole periods), V as the
// transposing read wants it (lane 4k + c of a 16-lane group points at token row k, columns 4c .. 4c + 3 of the group's 16;
// d-tile dt: ^ (dt % n) << 6, + whole periods).
template <int DQK, int DV>
struct Operands {
    using S = Shape<DQK, DV>;
    static constexpr int kXorBits = S::kKRow % 256 == 0 ? 4 : 3;              // chunk bits the K swizzle touches
    static constexpr int kPerXor = 1 << (kXorBits - 1);                      // contraction steps until those bits repeat
    static constexpr int kPerV = S::kVRow % 256 == 0 ? 4 : 2;                 // d-tiles until the address bits repeat
    int k_rd, v_rd;
    __device__ __forceinline__ Operands() {
        const int lane = static_cast<int>(threadIdx.x) & (kWave - 1), ln = lane & 31, lg = lane >> 5, l16 = lane >> 4, p16 = lane & 15;
        const int v_k = p16 >> 2, v_c4 = p16 & 3;
        k_rd = ln * S::kKRow + ((lg ^ k_swz<S::kKRow>(ln)) << 4);
        v_rd = S::kKBytes + (lg * 4 + v_k) * S::kVRow + ((((l16 & 1) * 2 + (v_c4 >> 1)) ^ v_swz<S::kVRow>(v_k)) << 4) + (v_c4 & 1) * 8;
    }
};

// Scores of the tile at LDS address `at`: register i of the result holds token (i/4)*8 + lg*4 + i%4, for this lane's row.
template <int DQK, int DV>
__device__ __forceinline__ f32x16 tile_scores(int at, const Operands<DQK, DV>& o, const bf16x8 (&q)[DQK / 16]) {
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const int ka = at + o.k_rd;
#pragma unroll
    for (int h = 0; h < DQK / 16; h += 4) {
        u32x4 kv[4];
        auto of = [&](int kk) { return (ka ^ ((kk % o.kPerXor) << 5)) + kk / o.kPerXor * (o.kPerXor * 32); };
        read_k4(kv, of(h), of(h + 1), of(h + 2), of(h + 3));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kv[kk]), q[h + kk], s, 0, 0, 0);
    }
    return s;
}

// -inf into the slots that this lane's row does not see, in a tile that begins rel > -32 tokens behind the first draft slot.
__device__ __forceinline__ void tile_mask(f32x16& s, uint64_t word, int rel) {
    uint32_t vis = rel >= 0 ? static_cast<uint32_t>(word >> rel) : (static_cast<uint32_t>(word << (-rel)) | ((1u << (-rel)) - 1u));
    vis >>= ((static_cast<int>(threadIdx.x) >> 5) & 1) * 4;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (!((vis >> ((i >> 2) * 8 + (i & 3))) & 1u)) s[i] = kNegInf;
}

// Scores -> pairs of probabilities, each a sum of TERMS bf16 terms, and the row's running maximum and sum.  Three terms hold all
// 24 bits of a probability, and the sum takes the fp32 value; one term is its rounding, and the sum takes that.
// With one term the reference is the tile's own maximum wherever that is within 8 of the highest so far (`top`): a tile's largest
// probability is then 1, which bf16 holds, as in a partition of that tile alone.
template <int TERMS>
__device__ __forceinline__ void tile_softmax(f32x16& s, float scale_log2, float& top, float& m_run, float& l_run, float& alpha, uint32_t (&term)[TERMS][8]) {
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    float m_use;
    if constexpr (TERMS > 1) {
        m_use = move_reference(mx, scale_log2, m_run, alpha);
    } else {
        mx = max_across_halves(mx) * scale_log2;
        const float m_new = mx > top - 8.f ? mx : m_run;
        top = fmaxf(top, mx);
        m_use = m_new == kNegInf ? 0.f : m_new;                // nothing visible yet: keep exp2 finite
        alpha = fast_exp2(m_run - m_use);
        m_run = m_new;
    }
    float psum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        s[i] = fast_exp2(fmaf(s[i], scale_log2, -m_use));
        s[i + 1] = fast_exp2(fmaf(s[i + 1], scale_log2, -m_use));
        if constexpr (TERMS > 1) psum += s[i] + s[i + 1];
        float r0 = s[i], r1 = s[i + 1];
#pragma unroll
        for (int k = 0; k < TERMS; ++k) {
            term[k][i >> 1] = cvt_pk_bf16(r0, r1);
            r0 -= bf16lo_to_f32(term[k][i >> 1]);              // (exact)
            r1 -= bf16hi_to_f32(term[k][i >> 1]);
        }
        if constexpr (TERMS == 1) psum = add_bf16_pair(term[0][i >> 1], psum);
    }
    l_run = l_run * alpha + psum;
}

// O^T[d][row] += V^T . (sum of the terms), from the tile at LDS address `at`.
template <int DQK, int DV, int TERMS>
__device__ __forceinline__ void tile_pv(int at, const Operands<DQK, DV>& o, const uint32_t (&term)[TERMS][8], f32x16 (&acc)[DV / 32]) {
    using S = Shape<DQK, DV>;
    const int va = at + o.v_rd;
    auto pair = [&](auto dtc) __attribute__((always_inline)) {
        constexpr int dt = decltype(dtc)::value, kPer = Operands<DQK, DV>::kPerV;
        u32x2 vr[2][4];
        read_v2<dt / kPer * (kPer * 64), 8 * S::kVRow>(vr, va ^ ((dt % kPer) << 6), va ^ (((dt + 1) % kPer) << 6));
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int d2 = 0; d2 < 2; ++d2) {
                const bf16x8 v = as_bf16x8(u32x4{vr[d2][2 * half][0], vr[d2][2 * half][1], vr[d2][2 * half + 1][0], vr[d2][2 * half + 1][1]});
#pragma unroll
                for (int k = 0; k < TERMS; ++k) {
                    const bf16x8 pk = as_bf16x8(u32x4{term[k][4 * half], term[k][4 * half + 1], term[k][4 * half + 2], term[k][4 * half + 3]});
                    acc[dt + d2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pk, acc[dt + d2], 0, 0, 0);
                }
            }
    };
    pair(std::integral_constant<int, 0>{});
    if constexpr (S::kDTiles >= 4) pair(std::integral_constant<int, 2>{});
    if constexpr (S::kDTiles >= 8) {
        pair(std::integral_constant<int, 4>{});
        pair(std::integral_constant<int, 6>{});
    }
}

// V rows with infinities or NaN, kept out of the product (bits of `left`: the tile's tokens): added to the rows that see the slot.
// row_of(token): that token's V row in the pool.
template <int TERMS, int DT, class RowOf>
__device__ __forceinline__ void tile_add_rows(uint32_t left, const uint32_t (&term)[TERMS][8], uint64_t word, int rel, f32x16 (&acc)[DT], RowOf&& row_of) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1), ln = lane & 31, lg = lane >> 5;
    for (; left; left &= left - 1) {
        const int j = __builtin_ctz(left), ij = (j >> 3) * 4 + (j & 3);
        float pj = 0.f;
#pragma unroll
        for (int k = TERMS - 1; k >= 0; --k) {
            uint32_t pair = term[k][0];                         // (a chain of selections: as a sum of masked words it cost the loop scalar registers)
#pragma unroll
            for (int i = 1; i < 8; ++i) {
                const uint32_t x = term[k][i];
                pair = (ij >> 1) == i ? x : pair;
            }
            pj += (ij & 1) ? bf16hi_to_f32(pair) : bf16lo_to_f32(pair);
        }
        pj = __shfl(pj, ln + ((j >> 2) & 1) * 32, kWave);                  // the half of the lanes that holds token j
        const bool sees = rel + j < 0 || ((word >> (rel + j)) & 1ull);
        const uint16_t* vrow = row_of(j);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const u32x2 v = *reinterpret_cast<const u32x2*>(vrow + dt * 32 + i4 * 8 + lg * 4);
                if (sees) {
                    acc[dt][i4 * 4] = fmaf(pj, bf16lo_to_f32(v[0]), acc[dt][i4 * 4]);
                    acc[dt][i4 * 4 + 1] = fmaf(pj, bf16hi_to_f32(v[0]), acc[dt][i4 * 4 + 1]);
                    acc[dt][i4 * 4 + 2] = fmaf(pj, bf16lo_to_f32(v[1]), acc[dt][i4 * 4 + 2]);
                    acc[dt][i4 * 4 + 3] = fmaf(pj, bf16hi_to_f32(v[1]), acc[dt][i4 * 4 + 3]);
                }
                __builtin_amdgcn_sched_barrier(0);   // (one load at a time: all of them in flight would spill)
            }
    }
}

// Which of a tile's V rows hold an infinity or NaN, as far as this thread's 16-byte chunks c = first, first + step, .. say (bits: tokens).
template <int DQK, int DV>
__device__ __forceinline__ uint32_t tile_nonfinite(const unsigned char* v_rows, int first, int step) {
    using S = Shape<DQK, DV>;
    uint32_t found = 0;
    for (int c = first; c < S::kVBytes / 16; c += step) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(v_rows + c * 16);
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if ((x[w] & 0x7f80u) == 0x7f80u || (x[w] & 0x7f800000u) == 0x7f800000u) found |= 1u << (c / (S::kVRow / 16));
    }
    return found;
}
// Clears the V rows of the tokens in `rows`.
template <int DQK, int DV>
__device__ __forceinline__ void tile_clear_rows(unsigned char* v_rows, uint32_t rows, int first, int step) {
    using S = Shape<DQK, DV>;
    for (int c = first; c < S::kVBytes / 16; c += step)
        if ((rows >> (c / (S::kVRow / 16))) & 1u) *reinterpret_cast<u32x4*>(v_rows + c * 16) = u32x4{0u, 0u, 0u, 0u};
}

}  // namespace tile

}  // namespace seer
