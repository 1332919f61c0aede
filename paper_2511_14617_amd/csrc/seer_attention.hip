// seer_verify_attention: entry point, device-side split-K plan, the general
// (any supported shape) partition kernel, and the split-K combine.
//
// What is computed (paper, Section 2.2: the target model verifies all draft
// tokens of a request in one pass, which beats serial decoding because the
// context is read from memory once instead of once per token): every one of the
// T = gamma + 1 verify slots of a request attends to the request's cached
// prefix and to the draft slots on its own root path (chain or multi-path tree,
// Section 3.4.2).  One read of a KV page must therefore serve all T slots and
// all G query heads that share the KV head.
#include "seer_attention.h"
#include "../../include/seer_verify_diag.h"

#include <stdio.h>

#include "seer_device.h"
#include "seer_plan_tables.h"

namespace seer {

// ---------------------------------------------------------------------------
// Plan: one workgroup turns ctx_len[B] into the tile line, the stretch of every
// partition workgroup and the partial slots of every request; a second one,
// beside it, compares neighbouring block-table rows (plan_shared_pages).  (Most calls of up to
// kSelfPlanRequests requests do without it: seer_plan.h.)
//
// The kernel is one dependent chain in front of every call that needs it, so it is
// written for the length of that chain: all global loads (lengths, header, shares of
// the speeds) are requested at once, one request and one stretch per thread, two
// exchanges between the waves for all sums and scans, and searches in LDS
// instead of walks over a request's pieces.  With 256 threads, four exchanges and
// walks it took 8.6 .. 12.5 us of every call; 4.9 with 75 to 110 requests (5.6 while it also smoothed the speeds).
// ---------------------------------------------------------------------------
constexpr int kPlanThreads = 1024;

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(AttnArgs p) {
    __shared__ PlanLds<kPlanThreads> lds;
    if (blockIdx.x == 1) plan_shared_pages(p, 0, p.B, kPlanThreads);
    else plan_tables<kPlanThreads>(p, lds);
}

// Which calls take whole requests (seer_attention_short.hip).  The host knows the table's width and not the lengths, and a model has one call that
// plans and many that reuse its plan: taken whole are the sizes where both kinds gain or stay level in the middle of all lengths, and where none
// makes a call slower by more than two microseconds.  39 500 random calls (tables of 32 ..
// 1536 tokens, 1 .. 1024 workgroups, 1 .. 128 rows, pages of 1 .. 64 tokens; all long, all short, any, or one long request among short ones), microseconds on the
// device of this kernel minus those of the partition kernels: median, 95th of 100 and worst of the calls that plan | of those that reuse (the same
// library against itself: 0, +0.2, +2.4 | 0, +0.2, +2.1).
//   heads of 64    up to 4 tiles -7.3 -6.4 -3.8 | -4.8 -3.8 -0.8; 16 tiles, 512 workgroups -6.1 -4.1 -3.0 | -3.4 -1.4 +0.5; 24 tiles, 256 workgroups
//                  -6.8 -2.9 -1.8 | -4.1 -0.3 +0.6; 32 tiles, 256 workgroups, up to 127 of them -3.2 -1.0 -0.8 | -1.1 +1.5 +1.7, more -11.0 -4.0 -1.9 | -7.5 -1.3 +1.0
//          not     more tiles -7.7 -0.7 +1.2 | -4.8 +1.7 +3.3; more workgroups -9.9 -0.6 +1.1 | -2.4 +3.4 +4.4
//   heads of 128   up to 4 tiles -8.1 -7.0 -5.3 | -4.9 -3.6 +0.3; 8 tiles, 512 workgroups -6.7 -5.1 -3.0 | -3.5 -2.2 +1.2; 16 tiles, 256 workgroups
//                  -5.1 -3.5 -2.8 | -2.2 -0.5 -0.3; 24 tiles, 256 workgroups, up to 31 of them -2.4 -1.5 -1.4 | +0.2 +1.3 +1.4, more -9.1 -3.1 -1.6 | -5.5 -0.3 +1.3
//          not     25 .. 32 tiles -10.1 -0.6 +0.4 | -6.0 +2.3 +3.1: a request of many tiles keeps its workgroup while others idle, and the partition
//                  kernels' stretches spread it (one as long as the table among short ones: 2048 tokens +6.6, 3072 +12.9); more workgroups, a second
//                  round of them, -11.2 -3.7 -1.7 | -4.3 +1.0 +4.0
//   192/128        up to 4 tiles, 256 workgroups -5.9 -4.3 -3.3 | -3.0 -1.3 -0.2; 8 tiles, 128 .. 256 workgroups -8.4 -4.2 -1.2 | -4.8 -1.4 +1.9
//          not     more workgroups -2.5 +1.7 +2.2 | +2.9 +5.4 +5.9; fewer of 5 .. 8 tiles -3.4 -1.1 -0.4 | -0.5 +2.1 +2.6; more tiles -6.2 +1.0 +2.2 | -2.8 +4.0 +8.1
//   256            up to 4 tiles, 256 workgroups: up to 32 rows -6.5 -4.6 -2.4 | -3.1 -1.2 +0.8, more rows from 65 workgroups on -6.1 -4.1 -2.9 | -2.8 -0.8 0.0
//          not     fewer of more rows, which share a tile's loads there, -3.6 -2.0 -0.7 | -0.1 +1.5 +2.6; 5 .. 8 tiles -8.4 -3.3 -0.2 | -4.9 -0.1 +3.4
// More than 64 rows of heads of 128 share a tile's loads in the kernel of the longer contexts.
bool short_call(const seer_attn_params& p) {
    if (!(gqa_layout(p) || tile_layout(p)) || p.max_splits == 1 || (p.flags & (SEER_ATTN_GENERAL_KERNEL | SEER_ATTN_STREAM_ONLY))) return false;
    const int rows = (p.Hq / p.Hkv) * p.T, tiles = short_tiles(p);
    if (rows > (p.Dqk == 128 ? 64 : 128) || static_cast<long long>(p.B) * p.max_pages_per_seq > kShortTableEntries) return false;
    struct Range {
        int Dqk, tiles, from, to;                   // tables of up to so many tiles: workgroups
    };
    static constexpr Range kRanges[] = {{64, 4, 1, 1024}, {64, 16, 1, 512}, {64, 32, 1, 256},
                                        {128, 4, 1, 1024}, {128, 8, 1, 512}, {128, 24, 1, 256},
                                        {192, 4, 1, 256}, {192, 8, 128, 256}, {256, 4, 1, 256}};
    const long long wgs = short_workgroups(p);
    for (const Range& r : kRanges)
        if (p.Dqk == r.Dqk && tiles <= r.tiles) return wgs >= (p.Dqk == 256 && rows > 32 ? 65 : r.from) && wgs <= r.to;
    return false;
}

hipError_t launch_plan(const AttnArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL(plan_kernel, dim3(2), dim3(kPlanThreads), 0, stream, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// General partition kernel: one workgroup per (stretch, query head, slot).
// Plain vector arithmetic, one KV token per wave iteration: lanes split the
// head dimension, the dot product is reduced with shuffles, the running
// (max, sum, acc) is kept per wave and the four waves are merged through LDS.
// Slow, but it covers every supported head size and page size, and serves as
// the on-device cross-check of the tiled kernels.
// ---------------------------------------------------------------------------
constexpr int kGenThreads = 256;
constexpr int kGenWaves = kGenThreads / kWave;

template <int DQK, int DV>
__global__ __launch_bounds__(kGenThreads) void attn_general_kernel(AttnArgs a) {
    constexpr int NQ = (DQK + 127) / 128;  // bf16 pairs per lane
    constexpr int NV = (DV + 127) / 128;
    if (static_cast<int>(blockIdx.x) >= a.wgs_per_head) return;       // (padding of the grid, see launch_general)
    const StretchRec rec = uniform_stretch(a, blockIdx.x);
    const int hq = blockIdx.y, t = blockIdx.z;
    const int kvh = hq / a.G;
    __shared__ float s_m[kGenWaves], s_l[kGenWaves];
    __shared__ float s_acc[kGenWaves][DV];
  const long long table_tok = static_cast<long long>(a.max_pages) * a.P;      // tokens that a row of the block table reaches
  const int max_tok = static_cast<int>(table_tok < 0x7fffffffLL ? table_tok : 0x7fffffffLL);
  int g = rec.tile_begin;
  for (int b = rec.b; b >= 0 && g < rec.tile_end; ++b) {
    const int t_lo = a.tile_off[b], t_hi = a.tile_off[b + 1];
    if (t_hi == t_lo) continue;
    const int n = a.ctx_len[b];
    const int piece_begin = (g - t_lo) * kPlanTile;
    const int piece_end = min(min(n, (min(rec.tile_end, t_hi) - t_lo) * kPlanTile), max_tok);   // (max_tok: n of a reused plan may be any)
    g = t_hi;
    const int item_idx = b + (a.balanced ? static_cast<int>(blockIdx.x) : 0);
    const int n0 = n - a.T;
    const uint64_t word = a.tree_mask ? a.tree_mask[static_cast<size_t>(b) * a.T + t]
                                      : (t >= 63 ? ~0ull : ((1ull << (t + 1)) - 1));
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const uint16_t* __restrict__ kp = static_cast<const uint16_t*>(a.k_pages);
    const uint16_t* __restrict__ vp = static_cast<const uint16_t*>(a.v_pages);
    const uint16_t* __restrict__ qrow =
        static_cast<const uint16_t*>(a.q) + ((static_cast<size_t>(b) * a.T + t) * a.Hq + hq) * DQK;

    float qlo[NQ], qhi[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int d = 2 * lane + 128 * i;
        const uint32_t pr = (d < DQK) ? *reinterpret_cast<const uint32_t*>(qrow + d) : 0u;
        qlo[i] = bf16lo_to_f32(pr);
        qhi[i] = bf16hi_to_f32(pr);
    }
    float m = kNegInf, l = 0.f;
    float alo[NV], ahi[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) alo[i] = ahi[i] = 0.f;

    const int32_t* __restrict__ table = a.block_table + static_cast<size_t>(b) * a.max_pages;
    bool bad_page = false;
    for (int j = piece_begin + wave; j < piece_end; j += kGenWaves) {
        const bool visible = (j < n0) || ((word >> (j - n0)) & 1ull);
        if (!visible) continue;  // uniform across the wave
        int page = table[j / a.P];
        if (page < 0 || page >= a.num_pages) {
            bad_page = true;
            page = min(max(page, 0), a.num_pages - 1);
        }
        const size_t tok = (static_cast<size_t>(page) * a.Hkv + kvh) * a.P + (j % a.P);
        const uint16_t* __restrict__ krow = kp + tok * DQK;
        float part = 0.f;
        uint32_t kpair[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int d = 2 * lane + 128 * i;
            kpair[i] = (d < DQK) ? *reinterpret_cast<const uint32_t*>(krow + d) : 0u;
            part = fmaf(qlo[i], bf16lo_to_f32(kpair[i]), part);
            part = fmaf(qhi[i], bf16hi_to_f32(kpair[i]), part);
        }
        const float s = wave_sum(part) * a.scale_log2;
        const float m_new = fmaxf(m, s);
        const float alpha = fast_exp2(m - m_new);
        const float p = fast_exp2(s - m_new);
        l = l * alpha + p;
        m = m_new;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int d = 2 * lane + 128 * i;
            uint32_t vpair;
            if (vp) vpair = (d < DV) ? *reinterpret_cast<const uint32_t*>(vp + tok * DV + d) : 0u;
            else vpair = (i < NQ) ? kpair[i < NQ ? i : 0] : 0u;  // shared latent: V = K[..., :DV]
            alo[i] = fmaf(p, bf16lo_to_f32(vpair), alo[i] * alpha);
            ahi[i] = fmaf(p, bf16hi_to_f32(vpair), ahi[i] * alpha);
        }
    }
    if (bad_page && lane == 0) atomicOr(&a.header->status, 2u);

    __syncthreads();                        // the previous piece's sums have been read
    if (lane == 0) {
        s_m[wave] = m;
        s_l[wave] = l;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int d = 2 * lane + 128 * i;
        if (d < DV) {
            s_acc[wave][d] = alo[i];
            s_acc[wave][d + 1] = ahi[i];
        }
    }
    __syncthreads();
    float M = s_m[0];
#pragma unroll
    for (int w = 1; w < kGenWaves; ++w) M = fmaxf(M, s_m[w]);
    float f[kGenWaves];
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < kGenWaves; ++w) {
        f[w] = (s_m[w] == kNegInf) ? 0.f : fast_exp2(s_m[w] - M);
        L += s_l[w] * f[w];
    }
    const size_t prow = (static_cast<size_t>(item_idx) * a.T + t) * a.Hq + hq;
    if (threadIdx.x == 0) {
        a.part_ml[2 * prow] = M;
        a.part_ml[2 * prow + 1] = L;
    }
    for (int d = threadIdx.x; d < DV; d += kGenThreads) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kGenWaves; ++w) v += s_acc[w][d] * f[w];
        a.part_acc[prow * DV + d] = v;
    }
  }  // pieces of the stretch
}

bool general_supports(int Dqk, int Dv) {
    return (Dqk == 64 && Dv == 64) || (Dqk == 128 && Dv == 128) || (Dqk == 256 && Dv == 256) ||
           (Dqk == 192 && Dv == 128) || (Dqk == 576 && Dv == 512);
}

hipError_t launch_general(const AttnArgs& a, hipStream_t stream) {
    // Of a short batch only the first few stretches hold work, for every head and slot: with a row of workgroups per (head, slot) that
    // is a multiple of 256 they would land on the same few CUs of each XCD row after row (2 requests of 4000 tokens, 17 slots, eight heads:
    // 217 us, 187 with rows of an odd multiple of 8; 16 of 1000, 9 slots, sixteen heads: 519, 480).
    const int row = a.wgs_per_head < 64 ? a.wgs_per_head : ((a.wgs_per_head + 7) / 8 | 1) * 8;
    const dim3 grid(row, a.Hq, a.T), block(kGenThreads);
#define SEER_GEN_CASE(DQK_, DV_)                                                                   \
    if (a.Dqk == DQK_ && a.Dv == DV_) {                                                            \
        hipLaunchKernelGGL((attn_general_kernel<DQK_, DV_>), grid, block, 0, stream, a);           \
        return hipGetLastError();                                                                  \
    }
    SEER_GEN_CASE(64, 64)
    SEER_GEN_CASE(128, 128)
    SEER_GEN_CASE(256, 256)
    SEER_GEN_CASE(192, 128)
    SEER_GEN_CASE(576, 512)
#undef SEER_GEN_CASE
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Combine: out = sum_s acc_s * 2^(m_s - M) / sum_s l_s * 2^(m_s - M), M = max_s m_s.
// A thread owns 4 consecutive output values of one row (16-byte loads of the fp32
// partials, one 8-byte bf16 store).  The kernel is a chain of memory round trips
// with few bytes per thread, so what counts is how many pieces are requested at
// once and that the chip is full: `slices` threads share the pieces of a row (slice
// i takes i, i + slices, ..), each requests up to eight pieces per round trip, and
// the slices are merged through LDS.  Measured against one thread per row that took
// four pieces at a time: requests of up to 128 pieces, 37 k threads of output (heads of
// 64) 16 -> 6 us; one KV head per GPU, up to 48 pieces 14.8 -> 7.9; 64 grouped requests
// (one slice) 13.9 -> 10.1; 86 MB of partials 34.8 -> 26.6 (3.2 TB/s).
// ---------------------------------------------------------------------------
constexpr int kCombineThreads = 256;

// Partial sums of one row slice: reference exponent, sum, four accumulators.
struct PartSum {
    float M, L;
    f32x4 v;
};

// Adds N pieces, all requested before the first is used (the ones past `n` re-read the last piece and count as having seen
// nothing).  ml / acc: the slice's first piece; strides in elements.
template <int N>
__device__ __forceinline__ void add_pieces(PartSum& s, const float2* ml, const float* acc, int n, size_t ml_stride, size_t acc_stride) {
    float2 msl[N];
    f32x4 p[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int su = min(u, n - 1);
        msl[u] = ml[su * ml_stride];
        p[u] = *reinterpret_cast<const f32x4*>(acc + su * acc_stride);
    }
    float M = s.M;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u >= n) msl[u].x = kNegInf;
        M = fmaxf(M, msl[u].x);
    }
    const float keep = s.M == kNegInf ? 0.f : fast_exp2(s.M - M);
    s.L *= keep;
#pragma unroll
    for (int c = 0; c < 4; ++c) s.v[c] = s.M == kNegInf ? 0.f : s.v[c] * keep;
    s.M = M;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        // a piece that saw nothing for this row (m = -inf) may hold anything in its accumulator
        const bool live = msl[u].x != kNegInf;
        const float w = live ? fast_exp2(msl[u].x - M) : 0.f;
        s.L += live ? msl[u].y * w : 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) s.v[c] += live ? p[u][c] * w : 0.f;
    }
}

// Requests whose shared pages one workgroup of the combine kernel counts: a thread's probes lie in 128 cache lines of their own (all 64
// requests of the tensor-parallel batch in one workgroup: 0.8 us of the call).
constexpr int kSharedRequests = 8;
inline int shared_pages_wgs(int B) { return (B + kSharedRequests - 1) / kSharedRequests; }

// What a call that plans leaves for the calls after it, by a workgroup of the combine kernel beside its others: the rates
// of the stretch indices from the partition kernel's measurements (in front of the partition kernel this was part of the plan
// kernel's chain), and, where the partition kernel planned for itself, the status word.
__device__ __forceinline__ void finish_call(const AttnArgs& a) {
    constexpr int kPer = kMaxWgsPerHead / kCombineThreads, kWaves = kCombineThreads / kWave;
    __shared__ float s_speed[kWaves], s_known[kWaves], s_rate[kWaves];
    __shared__ int s_status;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, W = a.wgs_per_head;
    const bool history = a.balanced && !a.fixed_split;
    if (tid == 0) s_status = 0;
    float est[kPer];
    float sum = 0.f, known = 0.f;
    if (history) {
        const bool valid = a.header->fb_magic == kFeedbackMagic && a.header->fb_w == W;
        uint32_t ticks[kPer], streamed[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int w = min(tid * kPer + k, W - 1);
            est[k] = a.fb_speed[w], ticks[k] = a.fb_time[w], streamed[k] = a.fb_tiles[w];
        }
        // relative speed of each stretch index (unknown: 0, also whatever a stale one held; the counters are this call's)
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (!valid) est[k] = 0.f;
            if (ticks[k] > 0u && streamed[k] > 0u) {
                const float meas = static_cast<float>(streamed[k]) / static_cast<float>(ticks[k]);
                est[k] = est[k] > 0.f ? 0.5f * est[k] + 0.5f * meas : meas;
            }
            if (!(est[k] > 0.f) || !(est[k] < 1e30f) || tid * kPer + k >= W) est[k] = 0.f;
            sum += est[k];
            known += est[k] > 0.f ? 1.f : 0.f;
        }
        sum = last_lane(wave_incl_scan(sum)), known = last_lane(wave_incl_scan(known));
        if (lane == 0) s_speed[wave] = sum, s_known[wave] = known;
    }
    bool bad_len = false, bad_page = false;
    if (a.self_plan) {
        if (tid < a.B) {
            const int n = a.ctx_len[tid];
            bad_len = n < a.T || n > a.max_ctx;
        }
        const int count = W * a.Hkv * a.row_blocks, waves = a.plan_waves;
        const uint64_t mask = waves >= 8 ? ~0ull : (1ull << (8 * waves)) - 1;
        uint64_t any = 0;
#pragma unroll 8
        for (int i = tid; i < count; i += kCombineThreads) any |= reinterpret_cast<const uint64_t*>(a.page_flags)[i] & mask;
        bad_page = any != 0;
    }
    __syncthreads();
    const int found = (__any(bad_len) ? 1 : 0) | (__any(bad_page) ? 2 : 0);
    if (found && lane == 0) atomicOr(&s_status, found);
    float rate[kPer], mine = 0.f, incl = 0.f;
    if (history) {
        sum = known = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += s_speed[w], known += s_known[w];
        const float mean = known > 0.f ? sum / known : 1.f;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            rate[k] = tid * kPer + k >= W ? 0.f : fminf(fmaxf(est[k] > 0.f ? est[k] / mean : 1.f, 0.75f), 4.f / 3.f);
            mine += rate[k];
        }
        incl = wave_incl_scan(mine);
        if (lane == kWave - 1) s_rate[wave] = incl;
    }
    __syncthreads();
    if (history) {
        float before = incl - mine, all = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) before += s_rate[w];
            all += s_rate[w];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int w = tid * kPer + k;
            if (w < W) {
                a.fb_before[w] = static_cast<uint32_t>(fminf(before / all, 0.99999994f) * 4294967296.f);
                before += rate[k];
                a.fb_speed[w] = est[k];
                a.fb_time[w] = 0u, a.fb_tiles[w] = 0u;
            }
        }
    }
    if (tid == 0) {
        if (history) a.header->fb_magic = kFeedbackMagic, a.header->fb_w = W;
        if (a.self_plan) a.header->status = static_cast<uint32_t>(s_status);
    }
}

// (five waves per SIMD: the extra workgroups' code must not cost the others theirs)
__global__ __launch_bounds__(kCombineThreads) __attribute__((amdgpu_waves_per_eu(5))) void combine_kernel(AttnArgs a, int blocks_per_request, int log2_slices, int log2_per_row,
                                                                  int extra) {
    __shared__ PartSum s_part[kCombineThreads];
    // the first workgroups (none in a call that reuses a plan): what is left for later calls
    if (static_cast<int>(blockIdx.x) < extra) {
        if (blockIdx.x == 0) finish_call(a);
        else plan_shared_pages(a, (blockIdx.x - 1) * kSharedRequests, min(static_cast<int>(blockIdx.x) * kSharedRequests, a.B), kCombineThreads);
        return;
    }
    const int block = static_cast<int>(blockIdx.x) - extra;
    const int b = block / blocks_per_request;
    const ReqSlots slots = a.req_slots[b];
    if (!has_plan(a)) return;
    const int per_b = a.T * a.Hq;
    const int tid = threadIdx.x;
    const int r = ((block - b * blocks_per_request) * kCombineThreads + tid) >> (log2_per_row + log2_slices);
    const int slice = (tid >> log2_per_row) & ((1 << log2_slices) - 1);
    const int d = (tid & ((1 << log2_per_row) - 1)) << 2;
    const bool row_ok = r < per_b;
    PartSum s{kNegInf, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
    int left = row_ok ? (slots.last - slots.first - slice + (1 << log2_slices)) >> log2_slices : 0;   // pieces of this slice
    if (left > 0) {
        const size_t at = static_cast<size_t>(slots.first + slice) * per_b + r;
        const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + at;
        const float* acc = a.part_acc + at * a.Dv + d;
        const size_t ml_stride = static_cast<size_t>(per_b) << log2_slices, acc_stride = ml_stride * a.Dv;
        while (left > 4) {
            add_pieces<8>(s, ml, acc, left, ml_stride, acc_stride);
            left -= 8;
            ml += 8 * ml_stride;
            acc += 8 * acc_stride;
        }
        if (left > 2) add_pieces<4>(s, ml, acc, left, ml_stride, acc_stride);
        else if (left > 0) add_pieces<2>(s, ml, acc, left, ml_stride, acc_stride);
    }
    if (log2_slices) {
        s_part[tid] = s;
        __syncthreads();
        if (slice || !row_ok) return;
        float M = s.M;
        for (int i = 1; i < (1 << log2_slices); ++i) M = fmaxf(M, s_part[tid + (i << log2_per_row)].M);
        PartSum sum{M, 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
        for (int i = 0; i < (1 << log2_slices); ++i) {
            const PartSum x = s_part[tid + (i << log2_per_row)];
            const float w = x.M == kNegInf ? 0.f : fast_exp2(x.M - M);
            sum.L += x.L * w;
#pragma unroll
            for (int c = 0; c < 4; ++c) sum.v[c] += x.M == kNegInf ? 0.f : x.v[c] * w;
        }
        s = sum;
    }
    if (!row_ok) return;
    const float inv = (s.L > 0.f) ? 1.f / s.L : 0.f;         // a row that saw nothing: zeros
    u32x2 o;
    o[0] = pack_bf16x2(s.v[0] * inv, s.v[1] * inv);
    o[1] = pack_bf16x2(s.v[2] * inv, s.v[3] * inv);
    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(a.out) + (static_cast<size_t>(b) * per_b + r) * a.Dv + d) = o;
}

// Threads that share the pieces of an output row: as many as fill the chip (about 2048 threads per CU) and fit a workgroup.
// Batches with a large output get one each: their requests are cut into few pieces and the chip is full anyway.
inline int combine_slices_log2(const AttnArgs& a, int log2_per_row) {
    const long long threads = static_cast<long long>(a.B) * a.T * a.Hq << log2_per_row;
    int s = 0;
    while (s < 4 && (threads << (s + 1)) <= kNumCU * 2048 && (2 << (s + log2_per_row)) <= kCombineThreads && (1 << s) < a.wgs_per_head) ++s;
    return a.balanced ? s : 0;
}

hipError_t launch_combine(const AttnArgs& a, hipStream_t stream) {
    const int log2_per_row = __builtin_ctz(static_cast<unsigned>(a.Dv >> 2));      // Dv is 64, 128, 256 or 512
    const int log2_slices = combine_slices_log2(a, log2_per_row);
    const long long threads = static_cast<long long>(a.T) * a.Hq << (log2_per_row + log2_slices);
    const int per_request = static_cast<int>((threads + kCombineThreads - 1) / kCombineThreads);
    const int extra = a.self_plan ? 1 + shared_pages_wgs(a.B) : (!a.reuse_plan && a.balanced && !a.fixed_split ? 1 : 0);
    hipLaunchKernelGGL(combine_kernel, dim3(static_cast<unsigned>(per_request) * static_cast<unsigned>(a.B) + extra), dim3(kCombineThreads),
                       0, stream, a, per_request, log2_slices, log2_per_row, extra);
    return hipGetLastError();
}

}  // namespace seer

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
namespace {

int validate_params(const seer_attn_params* p) {
    if (!p) return SEER_EINVAL;
    if (p->B < 0 || p->num_pages < 1 || p->max_pages_per_seq < 1 || p->page_size < 1) return SEER_EINVAL;
    if (p->T < 1 || p->T > SEER_MAX_T || p->Hq < 1 || p->Hkv < 1 || p->Hq % p->Hkv != 0) return SEER_ESHAPE;
    if (p->max_splits < 0 || p->max_splits > 256) return SEER_ESHAPE;
    if (p->flags & ~(SEER_ATTN_GENERAL_KERNEL | SEER_ATTN_FIXED_SPLIT | SEER_ATTN_STREAM_ONLY | SEER_ATTN_REUSE_PLAN))
        return SEER_EINVAL;
    if (p->Hq > 65535 || p->T * (int64_t)p->Hq * p->B > 0x7fffffffLL) return SEER_ESHAPE;
    if (!(p->scale > 0.f) || p->scale > 3.0e38f) return SEER_EINVAL;   // positive and finite
    if (!seer::general_supports(p->Dqk, p->Dv)) return SEER_EUNSUPPORTED;
    if (p->kv_shared_latent && p->Dv > p->Dqk) return SEER_ESHAPE;
    return SEER_OK;
}

}  // namespace

extern "C" size_t seer_verify_attention_workspace(const seer_attn_params* p) {
    if (validate_params(p) != SEER_OK || p->B == 0) return 0;
    return seer::workspace_layout(*p).total;
}

extern "C" size_t seer_verify_attention_status_offset(void) { return offsetof(seer::PlanHeader, status); }

extern "C" size_t seer_verify_attention_shared_tiles_offset(const seer_attn_params* p) {
    if (validate_params(p) != SEER_OK || p->B == 0) return 0;
    return seer::workspace_layout(*p).off_shared;
}

extern "C" const char* seer_verify_attention_kernel(const seer_attn_params* p) {
    if (validate_params(p) != SEER_OK) return nullptr;
    // the same tests, on the same fields, as the dispatch in run_verify_attention
    seer::AttnArgs a{};
    a.Dqk = p->Dqk, a.Dv = p->Dv, a.P = p->page_size, a.Hkv = p->Hkv;
    a.v_pages = p->kv_shared_latent ? nullptr : static_cast<const void*>(p);   // only null / non-null is looked at
    const bool tiled_ok = !(p->flags & SEER_ATTN_GENERAL_KERNEL);
    if (tiled_ok && seer::gqa128_supports(a)) {
        struct Names {
            char text[9][40], whole[3][80];
            Names() {
                for (int nw = 1; nw <= 8; ++nw)
                    snprintf(text[nw], sizeof(text[nw]), "attn_gqa128_kernel<%d,%d>", nw, seer::gqa_pipe_depth(nw));
                for (int nw = 1; nw <= 2; ++nw)                      // (no more than 64 rows)
                    snprintf(whole[nw], sizeof(whole[nw]), "%s; takes whole requests: attn_short_kernel<128,128>", text[nw]);
            }
        };
        static const Names names;
        const int rows = (p->Hq / p->Hkv) * p->T;
        if (seer::gqa_block_uses_helpers(seer::gqa_rows_per_block(rows))) return "attn_gqa128_kernel<4,2,helpers=4>";
        const int waves = seer::gqa_rows_per_block(rows) / 32;
        return seer::short_call(*p) ? names.whole[waves] : names.text[waves];
    }
    if (tiled_ok && seer::mla_supports(a)) return "attn_mla_kernel";
    if (seer::short_call(*p))
        return p->Dqk == 64 ? "attn_tile_kernel<64,64>; takes whole requests: attn_short_kernel<64,64>"
             : p->Dqk == 256 ? "attn_tile_kernel<256,256>; takes whole requests: attn_short_kernel<256,256>"
                             : "attn_tile_kernel<192,128>; takes whole requests: attn_short_kernel<192,128>";
    if (seer::tile_supports(*p))
        return p->Dqk == 64 ? "attn_tile_kernel<64,64>" : p->Dqk == 256 ? "attn_tile_kernel<256,256>" : "attn_tile_kernel<192,128>";
    if (p->Dqk == 64) return "attn_general_kernel<64,64>";
    if (p->Dqk == 128) return "attn_general_kernel<128,128>";
    if (p->Dqk == 256) return "attn_general_kernel<256,256>";
    if (p->Dqk == 192) return "attn_general_kernel<192,128>";
    return "attn_general_kernel<576,512>";
}

namespace {

int run_verify_attention(void* out, const void* q, const void* k_pages, const void* v_pages,
                         const int32_t* block_table, const int32_t* ctx_len, const uint64_t* tree_mask,
                         const seer_attn_params* p, void* workspace, size_t workspace_bytes, void* hip_stream,
                         hipEvent_t ev_begin, hipEvent_t ev_end) {
    const int rc = validate_params(p);
    if (rc != SEER_OK) return rc;
    if (p->B == 0) return SEER_OK;
    if (!out || !q || !k_pages || !block_table || !ctx_len) return SEER_EINVAL;
    if (p->kv_shared_latent ? (v_pages != nullptr) : (v_pages == nullptr)) return SEER_EINVAL;
    const seer::WorkspaceLayout w = seer::workspace_layout(*p);
    if (!workspace || workspace_bytes < w.total) return SEER_EWORKSPACE;
    auto misaligned = [](const void* ptr, uintptr_t a) { return reinterpret_cast<uintptr_t>(ptr) % a != 0; };
    if (misaligned(out, 16) || misaligned(q, 16) || misaligned(k_pages, 16) || misaligned(v_pages, 16) ||
        misaligned(workspace, 256) || misaligned(block_table, 4) || misaligned(ctx_len, 4) ||
        misaligned(tree_mask, 8))
        return SEER_EALIGN;

    char* ws = static_cast<char*>(workspace);
    seer::AttnArgs a{};
    a.out = out;
    a.q = q;
    a.k_pages = k_pages;
    a.v_pages = v_pages;
    a.block_table = block_table;
    a.ctx_len = ctx_len;
    a.tree_mask = tree_mask;
    a.header = reinterpret_cast<seer::PlanHeader*>(ws + w.off_header);
    a.req_slots = reinterpret_cast<const seer::ReqSlots*>(ws + w.off_slots);
    a.tile_off = reinterpret_cast<const int32_t*>(ws + w.off_tiles);
    a.stretch = reinterpret_cast<const seer::StretchRec*>(ws + w.off_stretch);
    a.balanced = w.max_splits > 1 ? 1 : 0;
    a.shared_tiles = reinterpret_cast<const int32_t*>(ws + w.off_shared);
    a.fb_time = reinterpret_cast<uint32_t*>(ws + w.off_fb);
    a.fb_tiles = a.fb_time + seer::kHistoryStride;
    a.fb_speed = reinterpret_cast<float*>(a.fb_tiles + seer::kHistoryStride);
    a.fb_before = reinterpret_cast<uint32_t*>(a.fb_speed + seer::kHistoryStride);
    a.inv_wgs = seer::reciprocal(w.wgs_per_head);
    a.inv_splits = seer::reciprocal(w.max_splits - 1);
    a.page_flags = reinterpret_cast<uint8_t*>(ws + w.off_flags);
    a.max_splits = w.max_splits;
    const long long max_ctx = static_cast<long long>(p->max_pages_per_seq) * p->page_size;
    a.max_ctx = max_ctx > 0x7fffffffLL - seer::kPlanTile ? 0x7fffffff - seer::kPlanTile : static_cast<int>(max_ctx);
    a.reuse_plan = (p->flags & SEER_ATTN_REUSE_PLAN) ? 1 : 0;
    a.self_plan = seer::self_plan_layout(*p) && !(p->flags & (SEER_ATTN_GENERAL_KERNEL | SEER_ATTN_REUSE_PLAN | SEER_ATTN_STREAM_ONLY)) ? 1 : 0;
    // (the shared-latent kernel records no speeds, and a single stretch is the whole line: nothing to keep a history of)
    a.fixed_split = (p->flags & SEER_ATTN_FIXED_SPLIT) || seer::mla_layout(*p) || w.wgs_per_head == 1 ? 1 : 0;
    a.stream_only = (p->flags & SEER_ATTN_STREAM_ONLY) ? 1 : 0;
    a.stream_partials = (w.total - w.off_acc) < seer::kStreamPartialsBelow ? 1 : 0;
    const bool tile_kernel = seer::tile_supports(*p);
    const int rows = (p->Hq / p->Hkv) * p->T;
    a.row_blocks = w.row_blocks;
    a.rows_per_block = tile_kernel ? seer::tile_rows_per_block(rows, p->Dqk) : seer::gqa_rows_per_block(rows);
    a.plan_waves = seer::mla_layout(*p) ? 4 : tile_kernel || !seer::gqa_block_uses_helpers(a.rows_per_block) ? a.rows_per_block / 32 : 8;
    a.part_ml = reinterpret_cast<float*>(ws + w.off_ml);
    a.part_acc = reinterpret_cast<float*>(ws + w.off_acc);
    a.B = p->B;
    a.T = p->T;
    a.Hq = p->Hq;
    a.Hkv = p->Hkv;
    a.G = p->Hq / p->Hkv;
    a.Dqk = p->Dqk;
    a.Dv = p->Dv;
    a.P = p->page_size;
    a.num_pages = p->num_pages;
    a.max_pages = p->max_pages_per_seq;
    a.wgs_per_head = w.wgs_per_head;
    a.scale_log2 = p->scale * seer::kLog2e;

    const bool tiled_ok = !(p->flags & SEER_ATTN_GENERAL_KERNEL);
    a.min_tiles = seer::tile_layout(*p) || seer::gqa_layout(*p) ? seer::kMinTiles : seer::kMinTilesLatent;
    a.fine_pieces = seer::gqa_layout(*p) ? static_cast<int32_t>(seer::kFinePartialsBelow / (sizeof(float) * p->T * p->Hq * p->Dv)) : 1 << 28;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (seer::short_call(*p)) {
        a.short_tiles = seer::short_tiles(*p), a.short_waves = seer::short_waves(p->Dqk, a.short_tiles);
        a.inv_pages = seer::reciprocal(p->max_pages_per_seq);
        a.self_plan = 0, a.fixed_split = 1;      // (no stretches are timed: the speed history stays as it is)
        hipError_t err = hipSuccess;
        if (ev_begin && (err = hipEventRecord(ev_begin, stream)) != hipSuccess) return static_cast<int>(err);
        if ((err = seer::launch_short(a, stream)) != hipSuccess) return static_cast<int>(err);
        if (ev_end && (err = hipEventRecord(ev_end, stream)) != hipSuccess) return static_cast<int>(err);
        return SEER_OK;
    }
    // the plan depends on the shape and on ctx_len only: the layers of one step can share it
    hipError_t err = a.reuse_plan || a.self_plan ? hipSuccess : seer::launch_plan(a, stream);
    if (err != hipSuccess) return static_cast<int>(err);
    if (ev_begin && (err = hipEventRecord(ev_begin, stream)) != hipSuccess) return static_cast<int>(err);
    if (tiled_ok && seer::gqa128_supports(a)) err = seer::launch_gqa128(a, stream);
    else if (tiled_ok && seer::mla_supports(a)) err = seer::launch_mla(a, stream);
    else if (tile_kernel) err = seer::launch_tile(a, stream);
    else err = seer::launch_general(a, stream);
    if (err != hipSuccess) return static_cast<int>(err);
    if (ev_end && (err = hipEventRecord(ev_end, stream)) != hipSuccess) return static_cast<int>(err);
    err = seer::launch_combine(a, stream);
    return err == hipSuccess ? SEER_OK : static_cast<int>(err);
}

}  // namespace

extern "C" int seer_verify_attention(void* out, const void* q, const void* k_pages, const void* v_pages,
                                     const int32_t* block_table, const int32_t* ctx_len,
                                     const uint64_t* tree_mask, const seer_attn_params* p, void* workspace,
                                     size_t workspace_bytes, void* hip_stream) {
    return run_verify_attention(out, q, k_pages, v_pages, block_table, ctx_len, tree_mask, p, workspace,
                                workspace_bytes, hip_stream, nullptr, nullptr);
}

extern "C" int seer_verify_attention_timed(void* out, const void* q, const void* k_pages, const void* v_pages,
                                           const int32_t* block_table, const int32_t* ctx_len,
                                           const uint64_t* tree_mask, const seer_attn_params* p,
                                           void* workspace, size_t workspace_bytes, void* hip_stream,
                                           void* event_begin, void* event_end) {
    if (!event_begin || !event_end) return SEER_EINVAL;
    return run_verify_attention(out, q, k_pages, v_pages, block_table, ctx_len, tree_mask, p, workspace,
                                workspace_bytes, hip_stream, static_cast<hipEvent_t>(event_begin),
                                static_cast<hipEvent_t>(event_end));
}

extern "C" const char* seer_strerror(int code) {
    switch (code) {
        case SEER_OK: return "ok";
        case SEER_EINVAL: return "null pointer or non-positive size";
        case SEER_ESHAPE: return "shape outside the supported range";
        case SEER_EUNSUPPORTED: return "no kernel for these head dimensions";
        case SEER_EWORKSPACE: return "workspace missing or too small";
        case SEER_EALIGN: return "pointer not aligned as required";
        case SEER_ELIMIT: return "problem larger than this fixed-size entry point holds";
        default: break;
    }
    if (code > 0) return hipGetErrorString(static_cast<hipError_t>(code));
    return "unknown seer error";
}
