// Tiled verify-attention partition kernel for grouped-query heads with
// D = 128 and pages of 16 (or a larger power of two) tokens (the shape of the paper's dense 8B- to 72B-class
// rollout models), on the gfx950 matrix cores.
//
// Why matrix cores although decoding is "memory bound": verification reads a
// KV page once for ALL T = gamma + 1 slots and all G heads of the group
// (Section 2.2: verifying n tokens in parallel beats n serial steps because
// memory is touched once).  That makes every 512 bytes of K+V feed G*T query
// rows (36 to 132 in the workloads here), i.e. 36-132 flop per byte: at HBM
// speed this is several hundred TFLOP/s, beyond the vector ALUs, so scores and
// P.V are MFMA contractions; everything else in this kernel exists to keep
// HBM streaming.
//
// Work decomposition
//   grid = (W, Hkv); workgroup (w, kv head) streams stretch w of the head's tile line
//   (see the plan in seer_attention.h) and, for each request the stretch touches,
//   handles all R = G*T query rows of that head.  Wave i owns rows [32i, 32i+32);
//   NW = ceil(R/32) waves per workgroup.
//
// Data flow per 32-token tile (two pages, 8 KB of K and 8 KB of V)
//   HBM -> LDS directly (global_load_lds_dwordx4: 16 bytes per lane, 1 KB per wave
//          instruction, no staging registers), into a ring of K slots and a ring of V slots,
//          D tiles in flight per workgroup while one is computed.  Rows are 256 B, unpadded;
//          the 16-byte chunks of a row are stored XOR-swizzled (the lane picks which
//          global chunk lands in its fixed LDS slot), which makes the operand reads
//          below free of bank conflicts.  Completion is tracked by hand: s_waitcnt
//          vmcnt(loads of the younger steps) then s_barrier.
//   S^T = K . Q^T    v_mfma_f32_32x32x16_bf16, M = tokens, N = rows, 8 steps over d;
//                    K operand = one ds_read_b128 per step, Q^T stays in 32 VGPRs
//   softmax          each lane owns ONE query row (N index = lane % 32) and 16 of the
//                    tile's 32 tokens, so max/sum are in-lane plus one cross-half
//                    exchange; the C registers of S^T are, as they stand, the
//                    B operand of the next product (no shuffle, no LDS round trip)
//   O^T += V^T . P^T M = d (4 tiles of 32), N = rows, 2 steps over the tokens; the
//                    V^T operand (8 tokens at one d) comes from the token-major tile
//                    through two transposing LDS reads (ds_read_b64_tr_b16)
//
// Software pipeline
//   A wave that ran a tile's three phases one after the other (scores on the matrix core,
//   softmax on the vector ALU, P.V on the matrix core) would leave each unit idle while the other
//   works, and waves sharing a SIMD would not fill each other's gaps either, because the per-tile
//   barrier keeps them in the same phase.  So one loop step works on three consecutive tiles,
//   with no dependence between the three parts:
//       step u:   P.V of tile u-2 (MFMA)  |  softmax of tile u-1 (VALU)  |  scores of tile u (MFMA)
//   K is needed two steps before the V of the same tile, hence the two rings (D+1 slots of 8 KB
//   each): step u issues the loads of K tile u+D and V tile u+D-2; both are consumed D steps
//   after they were issued, with the loads of D-1 steps in flight behind them.
//   The exponent reference of a row only moves when the new maximum exceeds it by more than 8
//   (in log2 units: the probabilities then stay below 2^8, as exact in bf16's 8 bits as values
//   below 1), which makes the rescaling of the 64 output accumulators rare.
#include <type_traits>
#include <utility>

#include "seer_attention.h"
#include "seer_device.h"
#include "seer_plan.h"
#include "seer_tile.h"

namespace seer {

constexpr int kD = 128;                  // head dim
constexpr int kMinPage = 16;             // tokens per page: 16, or a larger power of two (a 32-token tile is then inside one page)
constexpr int kTile = 32;                // tokens per tile
constexpr int kRowBytes = kD * 2;        // 256
constexpr int kKBytes = kTile * kRowBytes;   // 8192
static_assert(kTile == kPlanTile, "the plan counts work in tiles of this kernel");

// Swizzles: a row's 16-byte chunk c is stored at chunk position c ^ f(row).  LDS has 64 banks of
// 4 bytes (256 bytes per clock): a row is exactly one pass over the banks, so without a swizzle
// every row starts at bank 0.
//   K: f = row & 15        -> 16 consecutive rows, same chunk (one ds_read_b128 quarter-wave):
//                             16 distinct 16-byte bank groups
//   V: f = (row & 3) << 2  -> 4 consecutive rows, same 64-byte quarter of the row (half a wave of
//                             the transposing read): 4 distinct 64-byte groups
// (measured with several waves reading at once: these reach the rate of a linear access pattern,
// twice that of swizzles which only spread over 128 bytes)
__device__ __forceinline__ int k_swz(int row) { return row & 15; }
__device__ __forceinline__ int v_swz(int row) { return (row & 3) << 2; }

// Which waves issue the tile loads.  A direct-to-LDS load holds the issuing wave for about 27 ns (the
// vector memory path of a CU moves 64 bytes per clock), and with five waves on four SIMDs, waves 0 and 4
// share a SIMD and are the ones every step waits for: they are left out, waves 1..3 load.
template <int NW> struct Loaders { static constexpr int kFirst = 0, kCount = NW; };
template <> struct Loaders<5> { static constexpr int kFirst = 1, kCount = 3; };

// Cache policy of the tile loads: non-temporal.  A KV tile is used once per call by one workgroup, and
// streaming it (no allocation for reuse in the L2 and the memory-side cache) is what lets a gather of 4 KB
// blocks reach 6.9 TB/s on this part; the default policy tops out at 6.1 TB/s (bare read loops, plain loads
// and loads into LDS alike).
constexpr int kTileLoadPolicy = 2;   // the "nt" bit of the instruction's cache-policy field

// Loads of one half tile (K or V): its 8 one-KB blocks dealt round-robin to the loading waves.
template <int NW, int POLICY = kTileLoadPolicy>
__device__ __forceinline__ void issue_half_tile(unsigned char* slot, int wave, size_t p0, size_t p1,
                                                const unsigned char* base, int goff, bool is_k) {
    constexpr int NL = Loaders<NW>::kCount;
    const int li = wave - Loaders<NW>::kFirst;
    if (li < 0 || li >= NL) return;
#pragma unroll
    for (int i = 0; i < (8 + NL - 1) / NL; ++i) {
        const int j = li + i * NL;
        if (j < 8) {
            const size_t pg = (j < 4) ? p0 : p1;
            const int lane_off = is_k ? goff ^ ((j & 3) << 6) : goff;   // K rows 4j + l16: f = 4(j & 3) + l16
            const unsigned char* src = base + pg + (j & 3) * (4 * kRowBytes) + lane_off;
            __builtin_amdgcn_global_load_lds((const SEER_AS1 void*)(src), (SEER_AS3 void*)(slot + j * 1024), 16, 0, POLICY);
        }
    }
}

// 8 transposing reads: for each of the 4 d-tiles, the tokens +0..3 and +8..11 of one 16-token half.
// Within a 16-lane group, lane s = 4k + c points at token row k (of the 4 the group covers) and d
// columns 4c..4c+3 of the group's 16; lane i of the group receives the 4 tokens of column i.
// The reads are issued from an asm block that ends in its own s_waitcnt lgkmcnt(0): through the
// builtin, the compiler puts a vmcnt(0) in front of them (it cannot tell them apart from the
// direct-to-LDS loads still in flight), which would drain the ring on every tile.
#define SEER_GQA_TR8(vr_, a0_, a1_, a2_, a3_, OFF0, OFF1)                                                  \
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:" #OFF0 "\n"                                            \
                 "ds_read_b64_tr_b16 %1, %8 offset:" #OFF1 "\n"                                            \
                 "ds_read_b64_tr_b16 %2, %9 offset:" #OFF0 "\n"                                            \
                 "ds_read_b64_tr_b16 %3, %9 offset:" #OFF1 "\n"                                            \
                 "ds_read_b64_tr_b16 %4, %10 offset:" #OFF0 "\n"                                           \
                 "ds_read_b64_tr_b16 %5, %10 offset:" #OFF1 "\n"                                           \
                 "ds_read_b64_tr_b16 %6, %11 offset:" #OFF0 "\n"                                           \
                 "ds_read_b64_tr_b16 %7, %11 offset:" #OFF1 "\n"                                           \
                 "s_waitcnt lgkmcnt(0)"                                                                    \
                 : "=&v"(vr_[0][0]), "=&v"(vr_[0][1]), "=&v"(vr_[1][0]), "=&v"(vr_[1][1]), "=&v"(vr_[2][0]), \
                   "=&v"(vr_[2][1]), "=&v"(vr_[3][0]), "=&v"(vr_[3][1])                                    \
                 : "v"(a0_), "v"(a1_), "v"(a2_), "v"(a3_))

__device__ __forceinline__ void rescale_if_moved(f32x16 (&acc)[4], float alpha) {
    if (__any(alpha != 1.f)) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
    }
}

// One pipeline step at the ends of a piece, where not all three parts exist (the steady state is
// fused_step below).  k_off / v_off: byte offsets in LDS of the K slot the scores read and of the
// V slot (row part of the lane's address included) the P.V product reads.  alpha is the
// rescaling factor the previous step's softmax left for the output accumulators: it is applied
// before this step's P.V, and replaced by this step's softmax.
template <bool DO_QK, bool DO_SM, bool DO_PV, bool MASKED = true>
__device__ __forceinline__ void pipe_step(const unsigned char* lds, int k_off, int v_off, const int (&k_rd)[8],
                                          const int (&v_rd)[4], const bf16x8 (&qreg)[8], f32x16& s_sm,
                                          f32x16& s_qk, const uint32_t (&pk_pv)[8], uint32_t (&pk_sm)[8],
                                          f32x16 (&acc)[4], float& m_run, float& l_run, float& alpha,
                                          float scale_log2, uint32_t vis) {
    if constexpr (DO_PV) {
        rescale_if_moved(acc, alpha);
        alpha = 1.f;
        // O^T[d][row] += sum_token V[token][d] * P[row][token], 16 tokens at a time
        const int a0 = v_off + v_rd[0], a1 = v_off + v_rd[1], a2 = v_off + v_rd[2], a3 = v_off + v_rd[3];
        u32x2 vr[4][2];
        SEER_GQA_TR8(vr, a0, a1, a2, a3, 0, 2048);
        const bf16x8 pb0 = as_bf16x8(u32x4{pk_pv[0], pk_pv[1], pk_pv[2], pk_pv[3]});
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const bf16x8 va = as_bf16x8(u32x4{vr[dt][0][0], vr[dt][0][1], vr[dt][1][0], vr[dt][1][1]});
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb0, acc[dt], 0, 0, 0);
        }
        u32x2 vq[4][2];
        SEER_GQA_TR8(vq, a0, a1, a2, a3, 4096, 6144);
        const bf16x8 pb1 = as_bf16x8(u32x4{pk_pv[4], pk_pv[5], pk_pv[6], pk_pv[7]});
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const bf16x8 va = as_bf16x8(u32x4{vq[dt][0][0], vq[dt][0][1], vq[dt][1][0], vq[dt][1][1]});
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb1, acc[dt], 0, 0, 0);
        }
    }
    if constexpr (DO_QK) {
        // S^T[token][row] = sum_d K[token][d] * Q[row][d]
#pragma unroll
        for (int i = 0; i < 16; ++i) s_qk[i] = 0.f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 kv[4];
            const int b0 = k_off + k_rd[4 * h], b1 = k_off + k_rd[4 * h + 1], b2 = k_off + k_rd[4 * h + 2],
                      b3 = k_off + k_rd[4 * h + 3];
            asm volatile("ds_read_b128 %0, %4\n"
                         "ds_read_b128 %1, %5\n"
                         "ds_read_b128 %2, %6\n"
                         "ds_read_b128 %3, %7\n"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(kv[0]), "=&v"(kv[1]), "=&v"(kv[2]), "=&v"(kv[3])
                         : "v"(b0), "v"(b1), "v"(b2), "v"(b3));
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                s_qk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kv[kk]), qreg[4 * h + kk], s_qk, 0, 0, 0);
        }
    }
    if constexpr (DO_SM) {
        // register i of s_sm holds token (i/4)*8 + lg*4 + i%4 of the tile (vis is already shifted by lg*4)
        float mx = kNegInf;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if constexpr (MASKED)
                if (!((vis >> ((i >> 2) * 8 + (i & 3))) & 1u)) s_sm[i] = kNegInf;
            mx = fmaxf(mx, s_sm[i]);
        }
        const float m_use = move_reference(mx, scale_log2, m_run, alpha);
        float psum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = fast_exp2(fmaf(s_sm[i], scale_log2, -m_use));
            const float p1 = fast_exp2(fmaf(s_sm[i + 1], scale_log2, -m_use));
            pk_sm[i >> 1] = cvt_pk_bf16(p0, p1);
            psum = add_bf16_pair(pk_sm[i >> 1], psum);
        }
        l_run = l_run * alpha + psum;
    }
}

// Operand reads whose issue and completion are separated by hand.  The issuing block names the
// destination registers as outputs although they are only written when the read returns; the
// matching SEER_LGKM_WAIT block (s_waitcnt lgkmcnt(N), N = reads issued after the group: LDS
// returns in order) takes them as read-write operands, so every use of the data is ordered after
// the wait, and nothing between the two blocks has a reason to touch them.
#define SEER_TR8_ISSUE(vr_, a0_, a1_, a2_, a3_, OFF0, OFF1)                                                \
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%12\n"                                                  \
                 "ds_read_b64_tr_b16 %1, %8 offset:%13\n"                                                  \
                 "ds_read_b64_tr_b16 %2, %9 offset:%12\n"                                                  \
                 "ds_read_b64_tr_b16 %3, %9 offset:%13\n"                                                  \
                 "ds_read_b64_tr_b16 %4, %10 offset:%12\n"                                                 \
                 "ds_read_b64_tr_b16 %5, %10 offset:%13\n"                                                 \
                 "ds_read_b64_tr_b16 %6, %11 offset:%12\n"                                                 \
                 "ds_read_b64_tr_b16 %7, %11 offset:%13"                                                   \
                 : "=&v"(vr_[0][0]), "=&v"(vr_[0][1]), "=&v"(vr_[1][0]), "=&v"(vr_[1][1]), "=&v"(vr_[2][0]), \
                   "=&v"(vr_[2][1]), "=&v"(vr_[3][0]), "=&v"(vr_[3][1])                                    \
                 : "v"(a0_), "v"(a1_), "v"(a2_), "v"(a3_), "n"(OFF0), "n"(OFF1))
#define SEER_TR8_WAIT(N, vr_)                                                                              \
    asm volatile("s_waitcnt lgkmcnt(" #N ")"                                                               \
                 : "+v"(vr_[0][0]), "+v"(vr_[0][1]), "+v"(vr_[1][0]), "+v"(vr_[1][1]), "+v"(vr_[2][0]),    \
                   "+v"(vr_[2][1]), "+v"(vr_[3][0]), "+v"(vr_[3][1]))
#define SEER_K4_ISSUE(kv_, b0_, b1_, b2_, b3_, OFF)                                                        \
    asm volatile("ds_read_b128 %0, %4 offset:%8\n"                                                         \
                 "ds_read_b128 %1, %5 offset:%8\n"                                                         \
                 "ds_read_b128 %2, %6 offset:%8\n"                                                         \
                 "ds_read_b128 %3, %7 offset:%8"                                                           \
                 : "=&v"(kv_[0]), "=&v"(kv_[1]), "=&v"(kv_[2]), "=&v"(kv_[3])                              \
                 : "v"(b0_), "v"(b1_), "v"(b2_), "v"(b3_), "n"(OFF))
#define SEER_K4_WAIT(N, kv_)                                                                               \
    asm volatile("s_waitcnt lgkmcnt(" #N ")" : "+v"(kv_[0]), "+v"(kv_[1]), "+v"(kv_[2]), "+v"(kv_[3]))
#define SEER_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
// Keeps the computation of x in the block (and at the place) where it is written: a value whose
// only uses are in a later block is otherwise sunk there, out of the shadow of the MFMAs.
#define SEER_PIN(x) asm volatile("" : "+v"(x))

// The steady-state step: P.V of tile u-2 (8 MFMAs), scores of tile u (8 MFMAs) and the softmax of
// tile u-1 (about 80 vector-ALU instructions), with the instruction order fixed by hand: one
// MFMA, then the slice of softmax work that fits in the 32 cycles the matrix core is busy with
// it.  The compiler's scheduler, left alone, issues the sixteen MFMAs back to back and the
// softmax after them, which serialises the two units (a wave issues in order).  The operand
// reads run one group of four MFMAs ahead.
//
// issue_k / issue_v issue the step's HBM loads; they are called where their scalar address
// arithmetic runs in the shadow of LDS reads already issued and of MFMAs already queued.
//
// The slots read are at byte offsets K_IMM + k_off (K ring) and V_IMM + v_off (V ring, whose base is in v_rd); in the
// unrolled steady state the runtime parts are zero and the slot is an instruction immediate.
template <bool MASKED, int K_IMM, int V_IMM, typename IssueK, typename IssueV>
__device__ __forceinline__ void fused_step(int k_off, int v_off, const int (&k_rd)[8], const int (&v_rd)[4],
                                           const bf16x8 (&qreg)[8], f32x16& s_sm, f32x16& s_qk,
                                           const uint32_t (&pk_pv)[8], uint32_t (&pk_sm)[8], f32x16 (&acc)[4],
                                           float& m_run, float& l_run, float& alpha, float scale_log2,
                                           uint32_t vis, IssueK&& issue_k, IssueV&& issue_v) {
    const int a0 = v_off + v_rd[0], a1 = v_off + v_rd[1], a2 = v_off + v_rd[2], a3 = v_off + v_rd[3];
    u32x2 va[4][2], vb[4][2];
    u32x4 ka[4], kb[4];
    static_assert(K_IMM >= 0 && V_IMM >= 0 && K_IMM < 65536 && V_IMM + 6144 < 65536, "16-bit LDS offsets");
    SEER_TR8_ISSUE(va, a0, a1, a2, a3, V_IMM, V_IMM + 2048);
    SEER_TR8_ISSUE(vb, a0, a1, a2, a3, V_IMM + 4096, V_IMM + 6144);
    issue_k();
    rescale_if_moved(acc, alpha);
    if constexpr (MASKED) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (!((vis >> ((i >> 2) * 8 + (i & 3))) & 1u)) s_sm[i] = kNegInf;
    }
    SEER_TR8_WAIT(8, va);
    SEER_SCHED_FENCE();
    // ---- MFMAs 0..3: P.V on tokens 0..15 | row maximum
    const bf16x8 pb0 = as_bf16x8(u32x4{pk_pv[0], pk_pv[1], pk_pv[2], pk_pv[3]});
    float mx = kNegInf;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 v = as_bf16x8(u32x4{va[dt][0][0], va[dt][0][1], va[dt][1][0], va[dt][1][1]});
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pb0, acc[dt], 0, 0, 0);
        mx = fmaxf(fmaxf(mx, s_sm[4 * dt]), s_sm[4 * dt + 1]);
        mx = fmaxf(fmaxf(mx, s_sm[4 * dt + 2]), s_sm[4 * dt + 3]);
        SEER_PIN(mx);
        SEER_SCHED_FENCE();
    }
    {
        const int b0 = k_off + k_rd[0], b1 = k_off + k_rd[1], b2 = k_off + k_rd[2], b3 = k_off + k_rd[3];
        SEER_K4_ISSUE(ka, b0, b1, b2, b3, K_IMM);
    }
    issue_v();
    SEER_TR8_WAIT(4, vb);
    SEER_SCHED_FENCE();
    // ---- MFMAs 4..7: P.V on tokens 16..31 | exponent reference, first two pairs of probabilities
    const bf16x8 pb1 = as_bf16x8(u32x4{pk_pv[4], pk_pv[5], pk_pv[6], pk_pv[7]});
    float m_use = 0.f, psum = 0.f;
    // One pair of probabilities: scaled differences, exponentials, then the sum of the PREVIOUS pair (an
    // instruction that does not depend on the exponentials just issued, which need one more cycle before a
    // plain vector instruction may read them), then the packing of this pair.
    auto pair = [&](int i) __attribute__((always_inline)) {
        float p0 = fast_exp2(fmaf(s_sm[2 * i], scale_log2, -m_use));
        float p1 = fast_exp2(fmaf(s_sm[2 * i + 1], scale_log2, -m_use));
        asm volatile("" : "+v"(p0), "+v"(p1));
        if (i > 0) {
            psum = add_bf16_pair(pk_sm[i - 1], psum);
            SEER_PIN(psum);
        }
        pk_sm[i] = cvt_pk_bf16(p0, p1);
        SEER_PIN(pk_sm[i]);
    };
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 v = as_bf16x8(u32x4{vb[dt][0][0], vb[dt][0][1], vb[dt][1][0], vb[dt][1][1]});
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pb1, acc[dt], 0, 0, 0);
        if (dt == 0) {
            m_use = move_reference(mx, scale_log2, m_run, alpha);
            SEER_PIN(m_use);
            SEER_PIN(alpha);
            SEER_PIN(m_run);
        }
        if (dt == 2) pair(0);
        if (dt == 3) pair(1);
        SEER_SCHED_FENCE();
    }
    {
        const int b0 = k_off + k_rd[4], b1 = k_off + k_rd[5], b2 = k_off + k_rd[6], b3 = k_off + k_rd[7];
        SEER_K4_ISSUE(kb, b0, b1, b2, b3, K_IMM);
    }
    SEER_K4_WAIT(4, ka);
    SEER_SCHED_FENCE();
    // ---- MFMAs 8..15: scores of the next tile | the other six pairs
#pragma unroll
    for (int i = 0; i < 16; ++i) s_qk[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        s_qk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ka[kk]), qreg[kk], s_qk, 0, 0, 0);
        pair(2 + kk);
        SEER_SCHED_FENCE();
    }
    SEER_K4_WAIT(0, kb);
    SEER_SCHED_FENCE();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        s_qk = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kb[kk]), qreg[4 + kk], s_qk, 0, 0, 0);
        if (kk < 2) pair(6 + kk);
        if (kk == 2) {
            psum = add_bf16_pair(pk_sm[7], psum);
            l_run = l_run * alpha + psum;
            SEER_PIN(l_run);
        }
        SEER_SCHED_FENCE();
    }
}

// ---------------------------------------------------------------------------------------------------
// The helper shape: row blocks of 129 .. 144 rows (the multi-path tree on a group of four heads: 4 x 33 = 132).
//
// Four main waves hold the block's first 128 rows, 32 each, and a fifth wave for the rest would run the whole
// per-tile instruction stream for a handful of rows on a SIMD that a main wave needs.  So four helper waves double the
// main ones instead: a step works on a PAIR of tiles, the main waves on the even one, the helpers, with the same rows and
// a softmax state of their own, on the odd one.  Every SIMD has two independent instruction streams over a step, which is
// what hides operand reads, exponentials and the issue of tile loads; each wave runs the phases of its tile one after the
// other.  The leftover rows (at most 16) are one 16x16 product per 16 tokens: four of the eight waves, one per SIMD, take one
// half tile of the pair each (waves 0 and 1 the halves of the even tile, 6 and 7 those of the odd one) at the end of
// their step and at a raised issue priority; the other wave of the SIMD requests the tile loads, between its scores and its
// softmax: a direct-to-LDS load holds its wave for some 50 clocks, and with all eight waves requesting behind the barrier
// nothing else ran meanwhile (5 % of the kernel).
// At the end of a piece the two states of every row, and the four of a leftover row, become one through LDS, in a fixed order.
// Three pair slots of 32 KB: two pairs in flight while one is computed (three in flight: no change).
// What bounds it: the arithmetic alone takes 0.91 ms of the multi-path batch (128 requests, 1.37 M tokens, 132 rows), the
// load path alone 0.93 ms, both together 1.15 - 1.17 ms (1.19 - 1.22 with helpers that shared the leftover rows tile by
// tile beside a software-pipelined main wave).  Not kept: the helpers half a step behind the main waves (the second copy
// of the step spills, and a reload waits for the tile loads in flight).
// ---------------------------------------------------------------------------------------------------

// Pairs pay from this many tiles per piece on, five waves of the ordinary kernel are faster below: a short piece leaves half of
// its last pair idle, cannot fill the two pairs in flight and pays for the merge of the states like a long one.  Measured,
// whole call, five waves | pairs, by average tiles per piece: 3 tiles (44 requests of 80 tokens, two row blocks) 68.4 | 89.9 us, 10
// (128 of 500) 118.2 | 124.3, 18 (44 of 1000) 112.1 | 120.6, 28 (44 of 1500) 96.5 | 105.5, 35 (128 of 1400) 227.7 | 224.5, 39 (128 of
// 1500) 245.2 | 238.9, 77 (128 of 3000) 426.6 | 401.5.  Decided per stretch from its own pieces, so a batch of long and short
// requests uses both.
constexpr int kPairsFromTiles = 28;

namespace pairs {

constexpr int kWaves = 8, kSlots = 3;
constexpr int kTileBytes = 2 * kKBytes, kPairBytes = 2 * kTileBytes;          // a tile: K, then V
// end of a piece: four helper states of 32 rows (16 KB each), three of the leftover rows (8 KB each), their (m, l)
constexpr int kMergeMain = 0, kMergeLeft = 4 * 16384, kMergeMl = kMergeLeft + 3 * 8192, kMergeBytes = kMergeMl + 7 * kWave * 8;
constexpr int kLeftQ = kSlots * kPairBytes;                                  // the leftover rows' Q^T operands, [step][lane] x 16 bytes
constexpr int kLdsBytes = kLeftQ + 4096;
static_assert(kMergeBytes <= kSlots * kPairBytes, "the merge area fits the ring's memory");

typedef __attribute__((ext_vector_type(4))) short s16x4;

// Bits of a tile's 32 tokens that a row with mask word w sees; rel in (-32, 64): the tile's first token after the first slot.
__device__ __forceinline__ uint32_t visible(uint64_t w, int rel) {
    return rel >= 0 ? static_cast<uint32_t>(w >> rel) : (static_cast<uint32_t>(w << (-rel)) | ((1u << (-rel)) - 1u));
}

// One 16-token half of a tile for the leftover rows: this lane's row is p16, its tokens half * 16 + l16 * 4 + 0 .. 3.
// qa: LDS address of the lane's four Q^T operands (1 KB apart); ka: of the lane's K chunk (row half * 16 + p16, contraction steps 0 .. 3 by XOR with kk << 6);
// va: address of its transposing read (token row half * 16 + l16 * 4 + p16 / 4, d blocks 0 .. 7 by XOR with db << 5).
struct LeftState {
    f32x4 acc[8];
    float m, l;
};
__device__ __forceinline__ void left_half(LeftState& st, int qa, int ka, int va, float scale_log2, uint32_t vis) {
    u32x4 kv[4], q[4];
    const int k1 = ka ^ 64, k2 = ka ^ 128, k3 = ka ^ 192;
    asm volatile("ds_read_b128 %0, %8\n"
                 "ds_read_b128 %1, %9\n"
                 "ds_read_b128 %2, %10\n"
                 "ds_read_b128 %3, %11\n"
                 "ds_read_b128 %4, %12\n"
                 "ds_read_b128 %5, %12 offset:1024\n"
                 "ds_read_b128 %6, %12 offset:2048\n"
                 "ds_read_b128 %7, %12 offset:3072\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(kv[0]), "=&v"(kv[1]), "=&v"(kv[2]), "=&v"(kv[3]), "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
                 : "v"(ka), "v"(k1), "v"(k2), "v"(k3), "v"(qa));
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kv[kk]), as_bf16x8(q[kk]), s, 0, 0, 0);
    u32x2 vr[8];
    {
        const int a1 = va ^ 32, a2 = va ^ 64, a3 = va ^ 96, a4 = va ^ 128, a5 = va ^ 160, a6 = va ^ 192, a7 = va ^ 224;
        asm volatile("ds_read_b64_tr_b16 %0, %8\n"
                     "ds_read_b64_tr_b16 %1, %9\n"
                     "ds_read_b64_tr_b16 %2, %10\n"
                     "ds_read_b64_tr_b16 %3, %11\n"
                     "ds_read_b64_tr_b16 %4, %12\n"
                     "ds_read_b64_tr_b16 %5, %13\n"
                     "ds_read_b64_tr_b16 %6, %14\n"
                     "ds_read_b64_tr_b16 %7, %15\n"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(vr[0]), "=&v"(vr[1]), "=&v"(vr[2]), "=&v"(vr[3]), "=&v"(vr[4]), "=&v"(vr[5]), "=&v"(vr[6]), "=&v"(vr[7])
                     : "v"(va), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (!((vis >> i) & 1u)) s[i] = kNegInf;
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    float alpha;
    const float m_use = move_reference(mx, scale_log2, st.m, alpha);          // (takes the maximum over lane ^ 32 too)
    const float p0 = fast_exp2(fmaf(s[0], scale_log2, -m_use)), p1 = fast_exp2(fmaf(s[1], scale_log2, -m_use));
    const float p2 = fast_exp2(fmaf(s[2], scale_log2, -m_use)), p3 = fast_exp2(fmaf(s[3], scale_log2, -m_use));
    u32x2 pk;
    pk[0] = cvt_pk_bf16(p0, p1);
    pk[1] = cvt_pk_bf16(p2, p3);
    st.l = st.l * alpha + add_bf16_pair(pk[1], add_bf16_pair(pk[0], 0.f));
    if (__any(alpha != 1.f)) {
#pragma unroll
        for (int db = 0; db < 8; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) st.acc[db][i] *= alpha;
    }
    const s16x4 pb = __builtin_bit_cast(s16x4, pk);
#pragma unroll
    for (int db = 0; db < 8; ++db)
        st.acc[db] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vr[db]), pb, st.acc[db], 0, 0, 0);
}

// Scores of one tile for this lane's row (32 rows a wave), masked.  k: LDS address of the lane's K chunk of contraction step 0
// (step kk: ^ kk << 5); rel: first token of the tile relative to the first draft slot (uniform; masked slots have rel > -32).
__device__ __forceinline__ void scores(int k, const bf16x8 (&qreg)[8], f32x16& s, int rel, uint64_t word, int lg) {
    u32x4 ka[4], kb[4];
    {
        const int b1 = k ^ 32, b2 = k ^ 64, b3 = k ^ 96, b4 = k ^ 128, b5 = k ^ 160, b6 = k ^ 192, b7 = k ^ 224;
        SEER_K4_ISSUE(ka, k, b1, b2, b3, 0);
        SEER_K4_ISSUE(kb, b4, b5, b6, b7, 0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    SEER_K4_WAIT(4, ka);
    SEER_SCHED_FENCE();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ka[kk]), qreg[kk], s, 0, 0, 0);
    SEER_K4_WAIT(0, kb);
    SEER_SCHED_FENCE();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kb[kk]), qreg[4 + kk], s, 0, 0, 0);
    if (rel > -kTile) {
        const uint32_t vis = visible(word, rel) >> (lg * 4);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (!((vis >> ((i >> 2) * 8 + (i & 3))) & 1u)) s[i] = kNegInf;
    }
}

// Softmax of those scores and P.V.  The V^T operands (v: LDS address of the lane's transposing read, d-tile dt: ^ dt << 6) are
// requested before the exponentials and awaited after them.
__device__ __forceinline__ void softmax_pv(int v, f32x16& s, f32x16 (&acc)[4], float& m_run, float& l_run, float scale_log2) {
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 15; i += 2) mx = fmaxf(fmaxf(mx, s[i]), s[i + 1]);
    mx = fmaxf(mx, s[15]);
    float alpha;
    const float m_use = move_reference(mx, scale_log2, m_run, alpha);
    rescale_if_moved(acc, alpha);
    SEER_SCHED_FENCE();
    const int a1 = v ^ 64, a2 = v ^ 128, a3 = v ^ 192;
    u32x2 va[4][2], vb[4][2];
    SEER_TR8_ISSUE(va, v, a1, a2, a3, 0, 2048);
    SEER_TR8_ISSUE(vb, v, a1, a2, a3, 4096, 6144);
    float psum = 0.f;
    uint32_t pk[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float p0 = fast_exp2(fmaf(s[2 * i], scale_log2, -m_use));
        const float p1 = fast_exp2(fmaf(s[2 * i + 1], scale_log2, -m_use));
        pk[i] = cvt_pk_bf16(p0, p1);
        psum = add_bf16_pair(pk[i], psum);
    }
    l_run = l_run * alpha + psum;
    SEER_TR8_WAIT(8, va);
    SEER_SCHED_FENCE();
    const bf16x8 pb0 = as_bf16x8(u32x4{pk[0], pk[1], pk[2], pk[3]});
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(u32x4{va[dt][0][0], va[dt][0][1], va[dt][1][0], va[dt][1][1]}), pb0,
                                                          acc[dt], 0, 0, 0);
    SEER_TR8_WAIT(0, vb);
    SEER_SCHED_FENCE();
    const bf16x8 pb1 = as_bf16x8(u32x4{pk[4], pk[5], pk[6], pk[7]});
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(u32x4{vb[dt][0][0], vb[dt][0][1], vb[dt][1][0], vb[dt][1][1]}), pb1,
                                                          acc[dt], 0, 0, 0);
}

template <bool STREAM, bool STREAM_PARTIALS, bool SELF>
__device__ __forceinline__ void run(const AttnArgs& a, unsigned char* lds, const int* line, int kvh, int rb, int wg, const StretchRec& rec,
                                    bool new_history) {
    constexpr int NT = kWaves * kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ln = lane & 31, lg = lane >> 5, l16 = lane >> 4, p16 = lane & 15;
    const int set = wave >> 2, w4 = wave & 3;          // set 0 (main waves): even tiles, set 1 (helpers): odd tiles
    const bool has_left = wave < 2 || wave >= 6;       // one wave per SIMD; its 16-token half of its set's tile:
    const int half = wave & 1;

    int b = rec.b;
    const int slot_bias = a.balanced ? wg : 0;
    int g = rec.tile_begin;
    const int g_end = rec.tile_end;
    const uint64_t clock_begin = __builtin_amdgcn_s_memrealtime();
    bool bad_page = false;

    const unsigned char* __restrict__ kbase = static_cast<const unsigned char*>(a.k_pages);
    const unsigned char* __restrict__ vbase = static_cast<const unsigned char*>(a.v_pages);
    const int page_shift = __builtin_ctz(static_cast<unsigned>(a.P));
    const uint32_t page_bytes32 = static_cast<uint32_t>(a.Hkv) * a.P * kRowBytes;
    const size_t head_off = static_cast<size_t>(kvh) * a.P * kRowBytes;
    // tile loads: the four waves without leftover rows, two 1 KB blocks (eight rows) of K and of V of both tiles each
    const int loader = (wave + 2) & 3;
    const int row_in_half = (loader & 1) * 8;          // first row inside its 16-row half tile
    const int goff_k = (row_in_half + l16) * kRowBytes + ((p16 ^ k_swz(row_in_half + l16)) << 4);
    const int goff_k2 = (row_in_half + 4 + l16) * kRowBytes + ((p16 ^ k_swz(row_in_half + 4 + l16)) << 4);
    const int goff_v = (row_in_half + l16) * kRowBytes + ((p16 ^ v_swz(l16)) << 4);
    const int k_rd = ln * kRowBytes + ((lg ^ k_swz(ln)) << 4);
    const int v_k = p16 >> 2, v_c4 = p16 & 3;
    const int v_rd = (lg * 4 + v_k) * kRowBytes + ((((l16 & 1) * 2 + (v_c4 >> 1)) ^ v_swz(v_k)) << 4) + (v_c4 & 1) * 8;
    const int left_k = (half * 16 + p16) * kRowBytes + ((l16 ^ k_swz(p16)) << 4);
    const int left_v = (half * 16 + l16 * 4 + v_k) * kRowBytes + (((v_c4 >> 1) ^ v_swz(v_k)) << 4) + (v_c4 & 1) * 8;

    auto piece_words = [&](int bb) __attribute__((always_inline)) -> int {
        const int bc = min(bb, a.B - 1);
        const int32_t* ptr = a.tile_off + bc;
        if (lane == 1) ptr = a.tile_off + bc + 1;
        if (lane == 2) ptr = a.ctx_len + bc;
        if (lane == 3) ptr = a.shared_tiles + bc;
        return *ptr;
    };
    auto first_pages = [&](int bb, int page0) __attribute__((always_inline)) -> int {
        return (a.block_table + static_cast<size_t>(min(bb, a.B - 1)) * a.max_pages)[min(page0 + lane, a.max_pages - 1)];
    };
    int pw = SELF ? 0 : piece_words(b);
    int page_ahead = ((g - rec.req_begin) * kTile) >> page_shift;       // (see the kernel below)
    int pg_ahead = first_pages(b, page_ahead);
    int run_ahead = 0;                                 // SELF: how many of those a neighbouring request maps too
    if constexpr (SELF) run_ahead = shared_run(a, b, pg_ahead, neighbour_rows(a, b, page_ahead));
    const int g_first = g;

  for (; g < g_end; ++b) {
    if (SELF) pw = line_words(line, b);
    const int t_lo = __builtin_amdgcn_readlane(pw, 0), t_hi = __builtin_amdgcn_readlane(pw, 1);
    const int item_idx = b + slot_bias;
    const int n = __builtin_amdgcn_readlane(pw, 2);
    int shared_tiles = __builtin_amdgcn_readlane(pw, 3);
    const int pg_first = pg_ahead;
    const int page_first = page_ahead;
    NeighbourRows next_rows{0, 0};
    if constexpr (SELF) {
        if (run_ahead == kWave && t_hi > t_lo)
            run_ahead += shared_run_behind(a, b, page_first + kWave, (min(n, (min(g_end, t_hi) - t_lo) * kTile) - 1) >> page_shift);
        shared_tiles = static_cast<int>(static_cast<long long>(page_first + run_ahead) * a.P / kTile);
        next_rows = neighbour_rows(a, b + 1, 0);
    } else {
        pw = piece_words(b + 1);
    }
    pg_ahead = first_pages(b + 1, 0);
    page_ahead = 0;
    if (t_hi == t_lo) {
        if constexpr (SELF) run_ahead = shared_run(a, b + 1, pg_ahead, next_rows);
        continue;
    }
    const int tok_begin = (g - t_lo) * kTile;
    const int tok_end = min(n, (min(g_end, t_hi) - t_lo) * kTile);
    g = t_hi;
    const int n0 = n - a.T;
    const int n_tiles = (tok_end - tok_begin + kTile - 1) / kTile;
    const int n_pairs = (n_tiles + 1) >> 1;
    bare_barrier();                                    // every wave is done with the previous piece's slots

    const int R = min(a.G * a.T, (rb + 1) * a.rows_per_block);
    auto row_of = [&](int r, int& t, int& hq) __attribute__((always_inline)) -> bool {
        const bool ok = r < R;
        t = ok ? r / a.G : 0;
        hq = kvh * a.G + (ok ? r - t * a.G : 0);
        return ok;
    };
    auto mask_word = [&](int t, bool ok) __attribute__((always_inline)) -> uint64_t {
        uint64_t w = 0;
        if (ok) w = a.tree_mask ? a.tree_mask[static_cast<size_t>(b) * a.T + t] : (t >= 63 ? ~0ull : ((1ull << (t + 1)) - 1));
        return w;
    };
    int t, hq, t2, hq2;
    const bool row_ok = row_of(rb * a.rows_per_block + w4 * 32 + ln, t, hq);
    const bool left_ok = row_of(rb * a.rows_per_block + 128 + p16, t2, hq2) && has_left;
    uint64_t word = mask_word(t, row_ok), word2 = mask_word(t2, left_ok);
    u32x4 qv[8];
    {
        const uint16_t* qb = static_cast<const uint16_t*>(a.q) + static_cast<size_t>(b) * a.T * a.Hq * kD;
        const u32x4* qp = reinterpret_cast<const u32x4*>(qb + (static_cast<size_t>(t) * a.Hq + hq) * kD + lg * 8);
        const u32x4* qp2 = reinterpret_cast<const u32x4*>(qb + (static_cast<size_t>(t2) * a.Hq + hq2) * kD + l16 * 8);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            qv[kk] = u32x4{0u, 0u, 0u, 0u};
            if (row_ok) qv[kk] = qp[kk * 2];
        }
        if (wave == 0) {                               // (the four waves that serve these rows share one layout)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                u32x4 v = {0u, 0u, 0u, 0u};
                if (left_ok) v = qp2[kk * 4];
                *reinterpret_cast<u32x4*>(lds + kLeftQ + (kk * kWave + lane) * 16) = v;
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
        }
    }

    // page ids, 64 at a time, handed out with v_readlane (see the kernel below)
    const int32_t* __restrict__ table = a.block_table + static_cast<size_t>(b) * a.max_pages;
    const int last_page = (n - 1) >> page_shift;
    auto in_pool = [&](int pg, int idx) __attribute__((always_inline)) -> int {
        if (pg < 0 || pg >= a.num_pages) {
            if (idx <= last_page) bad_page = true;
            pg = min(max(pg, 0), a.num_pages - 1);
        }
        return pg;
    };
    int cache_base = page_first;
    int pg_cache = in_pool(pg_first, page_first + lane);
    // byte offset in a pool of the 16-row half of tile tb that holds this wave's block
    auto half_offset = [&](int tb) __attribute__((always_inline)) -> size_t {
        const int lp = tb >> page_shift;                 // 16-token pages: a tile is page lp (even) and lp + 1
        if (lp < cache_base || lp >= cache_base + kWave) {
            cache_base = lp;
            const int idx = cache_base + lane;
            pg_cache = in_pool(table[min(idx, a.max_pages - 1)], idx);
        }
        const int second = loader >> 1;                  // loaders 2 and 3 request rows 16 .. 31
        const int i = __builtin_amdgcn_readfirstlane(lp - cache_base + (a.P == kMinPage ? second : 0));
        const uint32_t pg = __builtin_amdgcn_readlane(pg_cache, i);
        const uint32_t in_page = static_cast<uint32_t>(tb + 16 * second) & (a.P - 1);
        return static_cast<uint64_t>(pg) * page_bytes32 + head_off + in_page * kRowBytes;
    };
    const int keep_until = shared_tiles - tok_begin / kTile;   // tiles below this index keep the default cache policy
    auto issue_pair = [&](int p) __attribute__((always_inline)) {
        const int slot_off = (p % kSlots) * kPairBytes;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int tile = 2 * p + s;
            if (tile < n_tiles) {
                const size_t off = half_offset(tok_begin + tile * kTile);
                unsigned char* dst = lds + slot_off + s * kTileBytes + loader * 2048;
                // through buffer descriptors of the 16 rows (scalar base, 32-bit lane offset): half the issue cost of the
                // form with 64-bit lane addresses, and fewer registers
                const __amdgpu_buffer_rsrc_t ks = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(kbase + off), 0, 16 * kRowBytes, 0x00020000);
                const __amdgpu_buffer_rsrc_t vs = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(vbase + off), 0, 16 * kRowBytes, 0x00020000);
                auto four = [&](auto policy) __attribute__((always_inline)) {
                    constexpr int POLICY = decltype(policy)::value;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ks, (SEER_AS3 void*)(dst), 16, goff_k, 0, 0, POLICY);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ks, (SEER_AS3 void*)(dst + 1024), 16, goff_k2, 0, 0, POLICY);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(vs, (SEER_AS3 void*)(dst + kKBytes), 16, goff_v, 0, 0, POLICY);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(vs, (SEER_AS3 void*)(dst + kKBytes + 1024), 16, goff_v, 1024, 0, POLICY);
                };
                if (tile < keep_until) four(std::integral_constant<int, 0>{});
                else four(std::integral_constant<int, kTileLoadPolicy>{});
            }
        }
    };
    if (!has_left) {
        issue_pair(0);
        if (n_pairs > 1) issue_pair(1);
    }

    bf16x8 qreg[8];
    {
        // the query rows and mask words have to have returned HERE (see the kernel below)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            asm volatile("" : "+v"(qv[kk]));
            qreg[kk] = as_bf16x8(qv[kk]);
        }
        asm volatile("" : "+v"(word), "+v"(word2));
        if (a.T < 64) word &= (1ull << a.T) - 1, word2 &= (1ull << a.T) - 1;
        if constexpr (SELF) {                          // (the next request's rows, requested in front of these, are there too)
            asm volatile("" : "+v"(pg_ahead), "+v"(next_rows.above), "+v"(next_rows.below));
            run_ahead = shared_run(a, b + 1, pg_ahead, next_rows);
        }
    }
    f32x16 acc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m_run = kNegInf, l_run = 0.f;
    LeftState left;
#pragma unroll
    for (int db = 0; db < 8; ++db) left.acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    left.m = kNegInf, left.l = 0.f;

    // top of step p: pair p has landed when at most the eight loads of pair p + 1 are outstanding
    auto step_top = [&](int p) __attribute__((always_inline)) {
        if (2 * p + 3 < n_tiles) wait_vmcnt<8>(); else wait_vmcnt<0>();
        bare_barrier();                                // ... for every wave, and every wave is done with step p - 1
        if (p == n_pairs - 1 && tok_begin + n_tiles * kTile > n) {
            // ragged last tile: clear the V rows past the end (0 * NaN must not reach the output)
            const int last = n_tiles - 1, first_bad = n - (tok_begin + last * kTile);
            unsigned char* vl = lds + (p % kSlots) * kPairBytes + (last & 1) * kTileBytes + kKBytes;
            for (int c = tid; c < kTile * 16; c += NT)
                if ((c >> 4) >= first_bad) *reinterpret_cast<u32x4*>(vl + c * 16) = u32x4{0u, 0u, 0u, 0u};
            __builtin_amdgcn_s_waitcnt(0xc07f);
            bare_barrier();
        }
        SEER_SCHED_FENCE();
    };
    if (has_left) __builtin_amdgcn_s_setprio(2);
    for (int p = 0; p < n_pairs; ++p) {
        step_top(p);
        const bool mine = 2 * p + set < n_tiles;
        const int rel = tok_begin + (2 * p + set) * kTile - n0;
        const int k_off = (p % kSlots) * kPairBytes + set * kTileBytes, v_off = k_off + kKBytes;
        if (!STREAM && mine) {
            f32x16 s;
            scores(k_off + k_rd, qreg, s, rel, word, lg);
            if (!has_left && p + 2 < n_pairs) issue_pair(p + 2);       // into the slot of pair p - 1
            softmax_pv(v_off + v_rd, s, acc, m_run, l_run, a.scale_log2);
        }
        if (has_left) {
            if (!STREAM && mine)
                left_half(left, kLeftQ + lane * 16, k_off + left_k, v_off + left_v, a.scale_log2,
                          rel <= -kTile ? ~0u : visible(word2, rel) >> (half * 16 + l16 * 4));
        } else if (STREAM && p + 2 < n_pairs) {
            issue_pair(p + 2);
        }
    }

    // ---- the helpers' states join the main waves' ------------------------------------------------------
    float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    float left_l = left.l + __shfl_xor(left.l, 32, kWave);
    left_l += __shfl_xor(left_l, 16, kWave);
    float2* ml = reinterpret_cast<float2*>(lds + kMergeMl);                      // [0..3]: helpers, [4..6]: leftover rows of waves 1, 6, 7
    bare_barrier();                                    // every wave has read the piece's last tiles
    if (set) {
        ml[w4 * kWave + lane] = float2{m_run, l_tot};
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4)
                *reinterpret_cast<f32x4*>(lds + kMergeMain + ((w4 * 16 + dt * 4 + i4) * kWave + lane) * 16) =
                    f32x4{acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
    }
    if (has_left && wave > 0) {
        const int o = wave == 1 ? 0 : wave - 5;
        ml[(4 + o) * kWave + lane] = float2{left.m, left_l};
#pragma unroll
        for (int db = 0; db < 8; ++db) *reinterpret_cast<f32x4*>(lds + kMergeLeft + ((o * 8 + db) * kWave + lane) * 16) = left.acc[db];
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    bare_barrier();
    auto store_partial = [&](float* dst, const f32x4& v) __attribute__((always_inline)) {
        if constexpr (STREAM_PARTIALS) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
        else *reinterpret_cast<f32x4*>(dst) = v;
    };
    if (!set) {
        const float2 other = ml[w4 * kWave + lane];
        const float M = fmaxf(m_run, other.x);
        const float f0 = m_run == kNegInf ? 0.f : fast_exp2(m_run - M), f1 = other.x == kNegInf ? 0.f : fast_exp2(other.x - M);
        const size_t prow = (static_cast<size_t>(item_idx) * a.T + t) * a.Hq + hq;
        if (row_ok && lg == 0) {
            a.part_ml[2 * prow] = M;
            a.part_ml[2 * prow + 1] = l_tot * f0 + other.y * f1;
        }
        float* __restrict__ po = a.part_acc + prow * kD + lg * 4;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                f32x4 v = *reinterpret_cast<const f32x4*>(lds + kMergeMain + ((w4 * 16 + dt * 4 + i4) * kWave + lane) * 16);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    v[c] = (f0 == 0.f ? 0.f : acc[dt][i4 * 4 + c] * f0) + (f1 == 0.f ? 0.f : v[c] * f1);
                if (row_ok) store_partial(po + dt * 32 + i4 * 8, v);
            }
    }
    if (wave == 0) {
        float mo[3], lo[3], M = left.m;
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            const float2 x = ml[(4 + o) * kWave + lane];
            mo[o] = x.x, lo[o] = x.y;
            M = fmaxf(M, x.x);
        }
        const float f = left.m == kNegInf ? 0.f : fast_exp2(left.m - M);
        float L = left_l * f, fo[3];
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            fo[o] = mo[o] == kNegInf ? 0.f : fast_exp2(mo[o] - M);
            L += lo[o] * fo[o];
        }
        const size_t prow = (static_cast<size_t>(item_idx) * a.T + t2) * a.Hq + hq2;
        if (left_ok && l16 == 0) {
            a.part_ml[2 * prow] = M;
            a.part_ml[2 * prow + 1] = L;
        }
        float* __restrict__ po = a.part_acc + prow * kD + l16 * 4;
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            f32x4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = f == 0.f ? 0.f : left.acc[db][c] * f;
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(lds + kMergeLeft + ((o * 8 + db) * kWave + lane) * 16);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] += fo[o] == 0.f ? 0.f : x[c] * fo[o];
            }
            if (left_ok) store_partial(po + db * 16, v);
        }
    }
  }  // pieces of the stretch
    if constexpr (SELF) publish_stretch(a, line, rec, wg, kvh, rb, wave, bad_page);
    else if (__any(bad_page) && lane == 0) atomicOr(&a.header->status, 2u);
    if (a.balanced && !a.fixed_split && tid == 0)
        record_speed(a, wg, kvh, rb, __builtin_amdgcn_s_memrealtime() - clock_begin, g_end - g_first, new_history);
}

}  // namespace pairs

template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// STREAM: diagnostic variant that keeps the whole load path (plan, page lookups, direct-to-LDS loads,
// waits, barriers, partial-result writes) and leaves out the arithmetic.  Its time is what the memory
// system allows for exactly this access pattern and launch shape: the ceiling the kernel's
// bytes-per-second should be read against.  It writes "saw nothing" partials, so the output is zero.
// STREAM_PARTIALS: the partial results leave with non-temporal stores (see kStreamPartialsBelow).
// NH: 0, or the three further waves that make five row waves into four main and four helper waves (see `pairs` above) in
// stretches whose pieces are long (kPairsFromTiles).
// SELF: every wave finds its stretch itself (seer_plan.h) instead of reading it from the plan kernel's tables.  (A template
// parameter: with both ways in one kernel the multi-path batch, which needs the tables, took 0.8 % longer through spilled scalars.)
template <int NW, int D, bool STREAM, bool STREAM_PARTIALS, int NH = 0, bool SELF = false>
__global__ __launch_bounds__((NW + NH) * kWave) __attribute__((amdgpu_waves_per_eu(NW + NH == 1 ? 1 : 2, 2)))
void attn_gqa128_kernel(AttnArgs a) {
    static_assert(NH == 0 || NW + NH == pairs::kWaves, "pairs need eight waves");
    constexpr int NT = NW * kWave;
    constexpr int NSLOT = D + 1;                    // slots in the K ring and in the V ring
    constexpr int NL = Loaders<NW>::kCount;        // waves that issue loads (the others have nothing to wait for)
    constexpr int CEIL = (8 + NL - 1) / NL;         // half-tile blocks of the busiest loading waves
    constexpr int FLOOR = 8 / NL;
    constexpr int REM = 8 % NL;                     // loaders below this index load CEIL blocks, the others FLOOR
    static_assert(D >= 1 && (D - 1) * 2 * CEIL < 64, "vmcnt range");

    // K ring, then V ring (pairs have a layout of their own)
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NH > 0 && pairs::kLdsBytes > 2 * NSLOT * kKBytes ? pairs::kLdsBytes : 2 * NSLOT * kKBytes];
    __shared__ int s_line[kLineWords];              // (see plan_stretch)
    constexpr int kVRing = NSLOT * kKBytes;

    // Workgroup ids are dealt round-robin to the 8 XCDs and dispatched in id order.  The grid is laid
    // out in groups of 8 stretches x Hkv heads so that the Hkv workgroups with the same stretch index
    // share XCD (id % 8) and dispatch round: the plan's per-index speed history relies on that.
    // The row blocks of a (stretch, head) are further workgroups with the same id % 8, so they share the XCD.
    int rest = blockIdx.x >> 3;
    const int kvh = rest % a.Hkv;
    rest /= a.Hkv;
    const int rb = rest % a.row_blocks;
    const int wg = (rest / a.row_blocks) * 8 + (blockIdx.x & 7);
    if (wg >= a.wgs_per_head) return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ln = lane & 31;
    const int lg = lane >> 5;
    const int l16 = lane >> 4;
    const int p16 = lane & 15;

    StretchRec rec;
    int pieces = 1;
    bool new_history = false;
    if (SELF) {
        const SelfPlan own = plan_stretch(a, s_line, wg);
        rec = own.rec, pieces = own.pieces, new_history = own.new_history;
        if (rec.b < 0) {
            publish_stretch(a, s_line, rec, wg, kvh, rb, wave, false);
            if (new_history && tid == 0) record_speed(a, wg, kvh, rb, 0, 0, true);
            return;
        }
    } else {
        rec = uniform_stretch(a, wg);
    }
    int b = rec.b;
    if constexpr (NH > 0) {
        // the pieces of this stretch: its requests up to the one the next stretch starts in (without it, if it starts with it)
        StretchRec next{-1, 0, 0, 0};
        if (!SELF) next = uniform_stretch(a, min(wg + 1, a.wgs_per_head - 1));
        if (b < 0) return;
        if (a.balanced && !SELF) {
            const int last = wg + 1 == a.wgs_per_head || next.b < 0 ? a.B - 1 : next.b - (next.req_begin == next.tile_begin ? 1 : 0);
            pieces = max(1, last - b + 1);
        }
        if (rec.tile_end - rec.tile_begin >= kPairsFromTiles * pieces) {
            pairs::run<STREAM, STREAM_PARTIALS, SELF>(a, lds, s_line, kvh, rb, wg, rec, new_history);
            return;
        }
        if (wave >= NW) {                           // (barriers wait for the waves that are left)
            if constexpr (SELF) publish_stretch(a, s_line, rec, wg, kvh, rb, wave, false);
            return;
        }
    } else {
        if (b < 0) return;
    }
    const int slot_bias = a.balanced ? wg : 0;
    int g = rec.tile_begin;
    const int g_end = rec.tile_end;
    const int g_first = g;
    const uint64_t clock_begin = __builtin_amdgcn_s_memrealtime();
    bool bad_page = false;

    const unsigned char* __restrict__ kbase = static_cast<const unsigned char*>(a.k_pages);
    const unsigned char* __restrict__ vbase = static_cast<const unsigned char*>(a.v_pages);
    const int page_shift = __builtin_ctz(static_cast<unsigned>(a.P));              // pages hold 2^page_shift tokens
    const uint32_t page_bytes32 = static_cast<uint32_t>(a.Hkv) * a.P * kRowBytes;   // one page, all kv heads
    const size_t head_off = static_cast<size_t>(kvh) * a.P * kRowBytes;
    const int goff_k0 = l16 * kRowBytes + ((p16 ^ k_swz(l16)) << 4);
    const int goff_v = l16 * kRowBytes + ((p16 ^ v_swz(l16)) << 4);
    int k_rd[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) k_rd[kk] = ln * kRowBytes + (((2 * kk + lg) ^ k_swz(ln)) << 4);
    const int v_k = p16 >> 2, v_c4 = p16 & 3, v_dhalf = l16 & 1;
    int v_rd[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        const int chunk = dt * 4 + v_dhalf * 2 + (v_c4 >> 1);
        // token lg*4 + k; the V ring's place behind the K ring is part of the lane address, so that the slot
        // offsets of both rings fit the 16-bit immediates of the LDS reads for rings of up to 8 slots
        v_rd[dt] = kVRing + (lg * 4 + v_k) * kRowBytes + ((chunk ^ v_swz(v_k)) << 4) + (v_c4 & 1) * 8;
    }

    // What a piece needs to know about its request comes from three small tables.  Read one after the other
    // (each value steers the next address or a branch) that is several dependent round trips to the L2 per
    // request boundary, several microseconds in which the workgroup has no tile in flight.  Instead one
    // vector load fetches all four words (lane i reads word i), and it is issued a whole piece ahead, together
    // with the first 64 page ids of that next request: by the time a piece ends, the next one's plan words
    // and page ids are in registers.
    auto piece_words = [&](int bb) __attribute__((always_inline)) -> int {
        const int bc = min(bb, a.B - 1);
        const int32_t* ptr = a.tile_off + bc;
        if (lane == 1) ptr = a.tile_off + bc + 1;
        if (lane == 2) ptr = a.ctx_len + bc;
        if (lane == 3) ptr = a.shared_tiles + bc;
        return *ptr;
    };
    auto first_pages = [&](int bb, int page0) __attribute__((always_inline)) -> int {
        return (a.block_table + static_cast<size_t>(min(bb, a.B - 1)) * a.max_pages)[min(page0 + lane, a.max_pages - 1)];
    };
    int pw = SELF ? 0 : piece_words(b);
    // 64 page ids of request b from page page_ahead on, where its next piece starts (a stretch starts inside a request, every
    // other piece at its request's first page)
    int page_ahead = ((g - rec.req_begin) * kTile) >> page_shift;
    int pg_ahead = first_pages(b, page_ahead);
    int run_ahead = 0;                                 // SELF: how many of those a neighbouring request maps too
    if constexpr (SELF) run_ahead = shared_run(a, b, pg_ahead, neighbour_rows(a, b, page_ahead));

  for (; g < g_end; ++b) {
    if (SELF) pw = line_words(s_line, b);
    const int t_lo = __builtin_amdgcn_readlane(pw, 0), t_hi = __builtin_amdgcn_readlane(pw, 1);
    const int item_idx = b + slot_bias;
    const int n = __builtin_amdgcn_readlane(pw, 2);
    int shared_tiles = __builtin_amdgcn_readlane(pw, 3);
    const int pg_first = pg_ahead;
    const int page_first = page_ahead;
    NeighbourRows next_rows{0, 0};
    if constexpr (SELF) {
        if (run_ahead == kWave && t_hi > t_lo)
            run_ahead += shared_run_behind(a, b, page_first + kWave, (min(n, (min(g_end, t_hi) - t_lo) * kTile) - 1) >> page_shift);
        shared_tiles = static_cast<int>(static_cast<long long>(page_first + run_ahead) * a.P / kTile);
        next_rows = neighbour_rows(a, b + 1, 0);
    } else {
        pw = piece_words(b + 1);          // in flight while this piece is worked on
    }
    pg_ahead = first_pages(b + 1, 0);
    page_ahead = 0;
    if (t_hi == t_lo) {
        if constexpr (SELF) run_ahead = shared_run(a, b + 1, pg_ahead, next_rows);
        continue;
    }
    const int tok_begin = (g - t_lo) * kTile;
    const int tok_end = min(n, (min(g_end, t_hi) - t_lo) * kTile);
    g = t_hi;
    const int n0 = n - a.T;
    const int n_tiles = (tok_end - tok_begin + kTile - 1) / kTile;
    bare_barrier();                                // every wave is done with the previous piece's slots

    const int R = min(a.G * a.T, (rb + 1) * a.rows_per_block);     // rows of this row block end here
    const int r = rb * a.rows_per_block + wave * 32 + ln;
    const bool row_ok = r < R;
    const int t = row_ok ? r / a.G : 0;
    const int hq = kvh * a.G + (row_ok ? r - t * a.G : 0);
    uint64_t word = 0;
    if (row_ok) {
        word = a.tree_mask ? a.tree_mask[static_cast<size_t>(b) * a.T + t]
                           : (t >= 63 ? ~0ull : ((1ull << (t + 1)) - 1));
    }
    // the query rows are requested here and awaited after the first tiles have been requested too
    bf16x8 qreg[8];
    u32x4 qv[8];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(
            static_cast<const uint16_t*>(a.q) + ((static_cast<size_t>(b) * a.T + t) * a.Hq + hq) * kD + lg * 8);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            qv[kk] = u32x4{0u, 0u, 0u, 0u};
            if (row_ok) qv[kk] = qp[kk * 2];
        }
    }

    f32x16 acc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m_run = kNegInf, l_run = 0.f, alpha = 1.f;

    // page ids, 64 at a time (lane l holds logical page cache_base + l), handed out with v_readlane.
    // With 16-token pages a tile is one even-numbered page and its successor, and windows start at even
    // pages, so one window test covers both; with larger pages a tile is 32 rows inside one page.
    const int32_t* __restrict__ table = a.block_table + static_cast<size_t>(b) * a.max_pages;
    const int last_page = (n - 1) >> page_shift;
    auto in_pool = [&](int pg, int idx) __attribute__((always_inline)) -> int {
        if (pg < 0 || pg >= a.num_pages) {
            if (idx <= last_page) bad_page = true;
            pg = min(max(pg, 0), a.num_pages - 1);
        }
        return pg;
    };
    // the window of page ids that the piece starts in has been fetched ahead
    int cache_base = page_first;
    int pg_cache = in_pool(pg_first, page_first + lane);
    auto page_pair = [&](int tb, size_t& p0, size_t& p1) __attribute__((always_inline)) {
        const int lp = tb >> page_shift;
        if (lp < cache_base || lp >= cache_base + kWave) {   // uniform
            cache_base = lp;
            const int idx = cache_base + lane;
            pg_cache = in_pool(table[min(idx, a.max_pages - 1)], idx);
        }
        const int i0 = __builtin_amdgcn_readfirstlane(lp - cache_base);
        const int i1 = a.P == kMinPage ? i0 + 1 : i0;
        const uint32_t g0 = __builtin_amdgcn_readlane(pg_cache, i0), g1 = __builtin_amdgcn_readlane(pg_cache, i1);
        const uint32_t in_page = static_cast<uint32_t>(tb & (a.P - 1));              // first row of the tile in its page
        p0 = static_cast<uint64_t>(g0) * page_bytes32 + head_off + in_page * kRowBytes;
        p1 = static_cast<uint64_t>(g1) * page_bytes32 + head_off + ((in_page + 16u) & (a.P - 1)) * kRowBytes;
    };

    // loads of step j: K tile j + D and V tile j + D - 2, where they exist.  The V tile sits in
    // the same pages of its pool as the K tile issued two steps earlier, whose offsets are kept.
    size_t pq0 = 0, pq1 = 0, pr0 = 0, pr1 = 0;     // page offsets of the K tiles of steps j - 1 and j - 2
    size_t pn0 = 0, pn1 = 0;
    // Tiles that a neighbouring request reads too (the plan's shared_tiles: a leading run of the request) are
    // loaded with the default cache policy, which keeps them in the memory-side cache for the repeats; all
    // other tiles are read once and stream past the caches.  The policy is an instruction immediate, so a
    // load site either streams or decides per tile with a scalar branch.
    const int keep_until = shared_tiles - tok_begin / kTile;   // tiles of this piece below this index are kept
    using StreamLoads = std::false_type;
    using CheckLoads = std::true_type;
    auto issue_k_at = [&](int kt, int slot_bytes, auto mode) __attribute__((always_inline)) {
        page_pair(tok_begin + kt * kTile, pn0, pn1);
        if (decltype(mode)::value && kt < keep_until)
            issue_half_tile<NW, 0>(lds + slot_bytes, wave, pn0, pn1, kbase, goff_k0, true);
        else
            issue_half_tile<NW>(lds + slot_bytes, wave, pn0, pn1, kbase, goff_k0, true);
    };
    auto issue_v_at = [&](int vt, int slot_bytes, auto mode) __attribute__((always_inline)) {
        if (decltype(mode)::value && vt < keep_until)
            issue_half_tile<NW, 0>(lds + kVRing + slot_bytes, wave, pr0, pr1, vbase, goff_v, false);
        else
            issue_half_tile<NW>(lds + kVRing + slot_bytes, wave, pr0, pr1, vbase, goff_v, false);
    };
    auto shift_pages = [&]() __attribute__((always_inline)) { pr0 = pq0, pr1 = pq1, pq0 = pn0, pq1 = pn1; };
    auto issue_k = [&](int j) __attribute__((always_inline)) {
        const int kt = j + D;
        if (kt < n_tiles) issue_k_at(kt, (kt % NSLOT) * kKBytes, CheckLoads{});
    };
    auto issue_v = [&](int j) __attribute__((always_inline)) {
        const int vt = j + D - 2;
        if (vt >= 0 && vt < n_tiles) issue_v_at(vt, (vt % NSLOT) * kKBytes, CheckLoads{});
        shift_pages();
    };
    auto issue_step = [&](int j) __attribute__((always_inline)) {
        issue_k(j);
        issue_v(j);
    };
    // The loads of step u - D have landed when at most the loads of the D - 1 steps after it are
    // outstanding.  That count is a compile-time number only while those steps all issued a full
    // K and V half tile; at the two ends of a piece wait for everything instead.
    auto wait_step = [&](int u) __attribute__((always_inline)) {
        const bool full = D > 1 && u >= 1 && u + D - 1 < n_tiles;
        if (full) {
            if (REM == 0 || wave - Loaders<NW>::kFirst < REM) wait_vmcnt<(D - 1) * 2 * CEIL>();
            else wait_vmcnt<(D - 1) * 2 * FLOOR>();
        } else {
            wait_vmcnt<0>();
        }
    };
    // visibility bits of tile j's 32 tokens for this lane's row, shifted to the lane's token half
    auto vis_of = [&](int j) __attribute__((always_inline)) -> uint32_t {
        const int rel = tok_begin + j * kTile - n0;          // uniform; in (-32, 64) for a masked tile
        if (rel <= -kTile) return ~0u;                        // a tile of prefix tokens only
        const uint32_t vis = rel >= 0 ? static_cast<uint32_t>(word >> rel)
                                      : (static_cast<uint32_t>(word << (-rel)) | ((1u << (-rel)) - 1u));
        return vis >> (lg * 4);
    };
    auto k_off = [&](int j) __attribute__((always_inline)) -> int { return (j % NSLOT) * kKBytes; };
    auto v_off = [&](int j) __attribute__((always_inline)) -> int {
        return (j % NSLOT) * kKBytes;              // (v_rd holds the ring's base)
    };

#pragma unroll
    for (int j = -D; j < 0; ++j) issue_step(j);
    {
        // Pin the point where the query rows and the mask word must have returned to HERE, before the tile
        // loop: left to itself the compiler waits for them at their first use inside the loop, with a wait
        // that also drains the direct-to-LDS loads of the tiles in flight, on every iteration.
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            asm volatile("" : "+v"(qv[kk]));
            qreg[kk] = as_bf16x8(qv[kk]);
        }
        uint32_t w_lo = static_cast<uint32_t>(word), w_hi = static_cast<uint32_t>(word >> 32);
        asm volatile("" : "+v"(w_lo), "+v"(w_hi));
        word = (static_cast<uint64_t>(w_hi) << 32) | w_lo;
        if (a.T < 64) word &= (1ull << a.T) - 1;
        if constexpr (SELF) {                          // (the next request's rows, requested in front of these, are there too)
            asm volatile("" : "+v"(pg_ahead), "+v"(next_rows.above), "+v"(next_rows.below));
            run_ahead = shared_run(a, b + 1, pg_ahead, next_rows);
        }
    }

    f32x16 s_a, s_b;
    uint32_t pk_a[8], pk_b[8];
#pragma unroll
    for (int i = 0; i < 16; ++i) s_a[i] = s_b[i] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) pk_a[i] = pk_b[i] = 0u;

    // Ragged last tile of a request: slots past the end hold whatever the page holds (NaN included), and
    // 0 * NaN must not reach the output: clear those V rows in LDS.  Every wave of the workgroup calls this at
    // step n_tiles + 1, after that step's barrier and before its P.V product.
    auto clear_ragged_tail = [&]() __attribute__((always_inline)) {
        const int tb = tok_begin + (n_tiles - 1) * kTile;
        if (tb + kTile > n) {
            unsigned char* vl = lds + kVRing + ((n_tiles - 1) % NSLOT) * kKBytes;
            const int first_bad = n - tb;
            int tid_here = tid;                    // (address computed here, not carried through the tile loop)
            asm volatile("" : "+v"(tid_here));
            for (int c = tid_here; c < kTile * 16; c += NT)
                if ((c >> 4) >= first_bad) *reinterpret_cast<u32x4*>(vl + c * 16) = u32x4{0u, 0u, 0u, 0u};
            __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0): the clears are done
            bare_barrier();
        }
    };

    // step 0: scores of tile 0 -> s_a
    wait_step(0);
    bare_barrier();
    issue_step(0);
    if constexpr (!STREAM)
        pipe_step<true, false, false>(lds, k_off(0), 0, k_rd, v_rd, qreg, s_b, s_a, pk_b, pk_a, acc, m_run, l_run, alpha,
                                      a.scale_log2, 0u);
    // step 1: softmax of tile 0 (s_a -> pk_a), scores of tile 1 -> s_b
    wait_step(1);
    bare_barrier();
    issue_step(1);
    {
        const uint32_t vis = vis_of(0);
        if constexpr (!STREAM) {
            if (n_tiles > 1)
                pipe_step<true, true, false>(lds, k_off(1), 0, k_rd, v_rd, qreg, s_a, s_b, pk_b, pk_a, acc, m_run,
                                             l_run, alpha, a.scale_log2, vis);
            else
                pipe_step<false, true, false>(lds, 0, 0, k_rd, v_rd, qreg, s_a, s_b, pk_b, pk_a, acc, m_run, l_run,
                                              alpha, a.scale_log2, vis);
        }
    }
    // steps 2 .. n_tiles - 1: P.V of tile u-2 (pk_a), softmax of tile u-1 (s_b -> pk_b), scores of tile u -> s_a,
    // after which the two register sets have swapped roles.  Tiles are masked from some tile on
    // (the draft slots are the last T positions), so the steps split into an unmasked run, taken
    // two steps per iteration so that the role swap costs no register moves, and a short masked run.
    auto full_step = [&](auto masked, int u, f32x16& s_sm, f32x16& s_qk, uint32_t (&pk_pv)[8],
                         uint32_t (&pk_sm)[8]) __attribute__((always_inline)) {
        wait_step(u);
        bare_barrier();                        // all waves: loads of step u - D landed, step u - 1 computed
        if constexpr (STREAM) {
            issue_k(u);
            issue_v(u);
        } else {
            fused_step<decltype(masked)::value, 0, 0>(
                k_off(u), v_off(u - 2), k_rd, v_rd, qreg, s_sm, s_qk, pk_pv, pk_sm, acc, m_run, l_run, alpha,
                a.scale_log2, decltype(masked)::value ? vis_of(u - 1) : 0u,
                [&]() __attribute__((always_inline)) { issue_k(u); },
                [&]() __attribute__((always_inline)) { issue_v(u); });
        }
    };
    auto swap_roles = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) { const float x = s_a[i]; s_a[i] = s_b[i]; s_b[i] = x; }
#pragma unroll
        for (int i = 0; i < 8; ++i) { const uint32_t x = pk_a[i]; pk_a[i] = pk_b[i]; pk_b[i] = x; }
    };
    {
        const int first_masked = n0 > tok_begin ? (n0 - tok_begin) / kTile : 0;   // first tile with masked slots
        const int u_split = min(max(first_masked + 1, 2), n_tiles);
        int u = 2;
        // Steady state proper: groups of P steps in which every load exists, every wait count is
        // the compile-time one, and (u = 2 mod NSLOT at the start of a group) every ring slot is
        // known at compile time.
        constexpr int P = NSLOT % 2 == 0 ? NSLOT : 2 * NSLOT;
        auto steady_step = [&](auto ic, auto mode) __attribute__((always_inline)) {
            constexpr int I = decltype(ic)::value;
            constexpr int kReadSlot = (2 + I) % NSLOT, kVReadSlot = I % NSLOT;
            constexpr int kIssueSlot = (1 + I) % NSLOT, kVIssueSlot = (I + NSLOT - 1) % NSLOT;
            if (REM == 0 || wave - Loaders<NW>::kFirst < REM) wait_vmcnt<(D - 1) * 2 * CEIL>();
            else wait_vmcnt<(D - 1) * 2 * FLOOR>();
            bare_barrier();
            const int uu = u + I;
            auto ik = [&]() __attribute__((always_inline)) { issue_k_at(uu + D, kIssueSlot * kKBytes, mode); };
            auto iv = [&]() __attribute__((always_inline)) {
                issue_v_at(uu + D - 2, kVIssueSlot * kKBytes, mode);
                shift_pages();
            };
            if constexpr (STREAM) {
                ik();
                iv();
            } else if constexpr (I % 2 == 0)
                fused_step<false, kReadSlot * kKBytes, kVReadSlot * kKBytes>(
                    0, 0, k_rd, v_rd, qreg, s_b, s_a, pk_a, pk_b, acc, m_run, l_run, alpha, a.scale_log2, 0u, ik, iv);
            else
                fused_step<false, kReadSlot * kKBytes, kVReadSlot * kKBytes>(
                    0, 0, k_rd, v_rd, qreg, s_a, s_b, pk_b, pk_a, acc, m_run, l_run, alpha, a.scale_log2, 0u, ik, iv);
        };
        auto steady_checking = [&](auto ic) __attribute__((always_inline)) { steady_step(ic, CheckLoads{}); };
        auto steady_streaming = [&](auto ic) __attribute__((always_inline)) { steady_step(ic, StreamLoads{}); };
        constexpr bool kUnrolled = NSLOT * kKBytes <= 65536;
        const int u_steady_end = min(u_split, n_tiles - D);
        // groups that may still load a kept tile (the oldest tile a group loads is V tile u + D - 2) decide per
        // tile; behind the kept run every load streams
        if constexpr (kUnrolled)
            for (; u + P <= u_steady_end && u + D - 2 < keep_until; u += P)
                for_each_index(steady_checking, std::make_integer_sequence<int, P>{});
        if constexpr (kUnrolled)
            for (; u + P <= u_steady_end; u += P) for_each_index(steady_streaming, std::make_integer_sequence<int, P>{});
        for (; u + 1 < u_split; u += 2) {
            full_step(std::false_type{}, u, s_b, s_a, pk_a, pk_b);
            full_step(std::false_type{}, u + 1, s_a, s_b, pk_b, pk_a);
        }
        if (u < u_split) {
            full_step(std::false_type{}, u, s_b, s_a, pk_a, pk_b);
            swap_roles();
            ++u;
        }
        for (; u < n_tiles; ++u) {
            full_step(std::true_type{}, u, s_b, s_a, pk_a, pk_b);
            swap_roles();
        }
    }
    // now: s_b = scores of the last tile (if n_tiles > 1), pk_a = probabilities of tile n_tiles - 2
    if (n_tiles > 1) {
        const int u = n_tiles;
        wait_step(u);
        bare_barrier();
        issue_step(u);
        if constexpr (!STREAM)
            pipe_step<false, true, true>(lds, 0, v_off(u - 2), k_rd, v_rd, qreg, s_b, s_a, pk_a, pk_b, acc, m_run, l_run,
                                         alpha, a.scale_log2, vis_of(u - 1));
#pragma unroll
        for (int i = 0; i < 8; ++i) pk_a[i] = pk_b[i];
    }
    {
        const int u = n_tiles + 1;
        wait_step(u);
        bare_barrier();
        clear_ragged_tail();
        if constexpr (!STREAM)
            pipe_step<false, false, true>(lds, 0, v_off(n_tiles - 1), k_rd, v_rd, qreg, s_b, s_a, pk_a, pk_b, acc, m_run,
                                          l_run, alpha, a.scale_log2, 0u);
    }

    // ---- partial result: (reference exponent, sum, unnormalised O) per row ------------
    float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    if (row_ok && lg == 0) {
        const size_t prow = (static_cast<size_t>(item_idx) * a.T + t) * a.Hq + hq;
        a.part_ml[2 * prow] = m_run;
        a.part_ml[2 * prow + 1] = l_tot;
    }
    auto store_partial = [&](float* dst, const f32x4& v) __attribute__((always_inline)) {
        // (a compile-time choice: in two arms of a run-time branch the compiler folds the two stores of the
        // same value into one plain store)
        if constexpr (STREAM_PARTIALS) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
        else *reinterpret_cast<f32x4*>(dst) = v;
    };
    if constexpr (NW <= 2 && NW * 16384 <= 2 * NSLOT * kKBytes) {
        // The accumulators hold, per lane, 16-byte pieces of a row that lie 32 bytes apart; written out as they
        // are, one store instruction touches 32 rows with 32 bytes each.  Through the ring (free now: 16 KB per
        // wave, 16-byte chunks XORed with the row so that neither side has bank conflicts) every store
        // instruction writes two whole rows of 512 bytes.  Worth 0.6 % of the kernel on the memory-bound
        // two-wave shape (many short pieces); nothing measurable with three waves and more, which keep the
        // direct stores.
        bare_barrier();                                  // every wave has read the last tiles
        unsigned char* st = lds + wave * 16384;
        // (the addresses below are computed here, from a copy of the lane index the compiler cannot see through:
        // hoisted out of the piece loop they would hold registers through the tile loop, which has none to spare)
        int ln_here = ln;
        asm volatile("" : "+v"(ln_here));
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 v = {acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
                const int c = dt * 8 + i4 * 2 + lg;
                *reinterpret_cast<f32x4*>(st + ln_here * 512 + ((c ^ ln_here) << 4)) = v;
            }
        const int first_row = rb * a.rows_per_block + wave * 32;
#pragma unroll 2
        for (int k = 0; k < 16; ++k) {                   // (not unrolled further: sixteen rows in flight spill registers)
            const int rr = 2 * k + lg;                   // row of the wave; this lane moves chunk ln of it
            const f32x4 v = *reinterpret_cast<const f32x4*>(st + rr * 512 + ((ln_here ^ rr) << 4));
            const int r2 = first_row + rr;
            if (r2 < R) {
                const int t2 = r2 / a.G;
                const int hq2 = kvh * a.G + (r2 - t2 * a.G);
                const size_t prow = (static_cast<size_t>(item_idx) * a.T + t2) * a.Hq + hq2;
                store_partial(a.part_acc + prow * kD + ln * 4, v);
            }
        }
    } else if (row_ok) {
        int lg_here = lg;                                // (as above)
        asm volatile("" : "+v"(lg_here));
        const size_t prow = (static_cast<size_t>(item_idx) * a.T + t) * a.Hq + hq;
        float* __restrict__ po = a.part_acc + prow * kD + lg_here * 4;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 v = {acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
                store_partial(po + dt * 32 + i4 * 8, v);
            }
    }
  }  // pieces of the stretch
    if constexpr (SELF) publish_stretch(a, s_line, rec, wg, kvh, rb, wave, bad_page);
    else if (__any(bad_page) && lane == 0) atomicOr(&a.header->status, 2u);
    // speed history for the next call's plan: tiles streamed and time taken, by stretch index
    if (a.balanced && !a.fixed_split && tid == 0)
        record_speed(a, wg, kvh, rb, __builtin_amdgcn_s_memrealtime() - clock_begin, g_end - g_first, new_history);
}

bool gqa128_supports(const AttnArgs& a) {
    return a.Dqk == kD && a.Dv == kD && a.P >= kMinPage && a.P <= 1024 && (a.P & (a.P - 1)) == 0 &&
           a.v_pages != nullptr && a.Hkv <= 65535;
}

hipError_t launch_gqa128(const AttnArgs& a, hipStream_t stream) {
    const int nw = a.rows_per_block / 32;
    const dim3 grid(static_cast<unsigned>((a.wgs_per_head + 7) / 8) * 8u * static_cast<unsigned>(a.Hkv) *
                    static_cast<unsigned>(a.row_blocks));
    const dim3 block((gqa_block_uses_helpers(a.rows_per_block) ? 8 : nw) * kWave);
#define SEER_GQA_LAUNCH(NW_, NH_)                                                                                       \
    do {                                                                                                              \
        constexpr int D_ = gqa_pipe_depth(NW_);                                                                       \
        if (a.stream_only && a.stream_partials) hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, true, true, NH_>), grid, block, 0, stream, a);   \
        else if (a.stream_only) hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, true, false, NH_>), grid, block, 0, stream, a);                  \
        else if (a.self_plan && a.stream_partials) hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, false, true, NH_, true>), grid, block, 0, stream, a); \
        else if (a.self_plan) hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, false, false, NH_, true>), grid, block, 0, stream, a);             \
        else if (a.stream_partials) hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, false, true, NH_>), grid, block, 0, stream, a);              \
        else hipLaunchKernelGGL((attn_gqa128_kernel<NW_, D_, false, false, NH_>), grid, block, 0, stream, a);                                    \
    } while (0)
    // 129 .. 144 query rows in a row block: five waves, or four main waves and four helpers
    if (gqa_block_uses_helpers(a.rows_per_block)) {
        SEER_GQA_LAUNCH(5, 3);
        return hipGetLastError();
    }
    switch (nw) {
        case 1: SEER_GQA_LAUNCH(1, 0); break;
        case 2: SEER_GQA_LAUNCH(2, 0); break;
        case 3: SEER_GQA_LAUNCH(3, 0); break;
        case 4: SEER_GQA_LAUNCH(4, 0); break;
        case 5: SEER_GQA_LAUNCH(5, 0); break;
        case 6: SEER_GQA_LAUNCH(6, 0); break;
        case 7: SEER_GQA_LAUNCH(7, 0); break;
        case 8: SEER_GQA_LAUNCH(8, 0); break;
        default: return hipErrorInvalidValue;
    }
#undef SEER_GQA_LAUNCH
    return hipGetLastError();
}

}  // namespace seer
