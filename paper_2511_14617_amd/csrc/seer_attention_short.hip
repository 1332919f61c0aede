// Verify attention of whole requests, for block tables that hold short contexts only: one workgroup takes all tokens of a request
// for 32 query rows of a KV head, its waves share the tokens, and they merge in LDS.  One kernel, no partial results in memory
// and no combine kernel.  Separate K and V pools, all head sizes of the tiled kernels.
//
// What bounds it: the length of its chain (launch, page ids, one tile's loads after the other, the merge), not a roofline.  The
// partition kernels cut a short batch into stretches of a tile or two to fill the chip; what they save in tiles per workgroup
// they spend on partial results and on the combine kernel behind them.  Here a tile belongs to one wave from its loads to its
// product, in LDS of that wave's own, so there is no barrier until the merge; the K rows of a wave's next tile are requested
// behind the scores, the V rows behind the product.  A CU holds twelve tiles of heads of 64 (three workgroups of four waves; eight
// where a workgroup has eight), eight of heads of 128, seven or four of 192/128 (one workgroup of as many waves), four of heads of 256.
//
// The workgroups in front of the grid leave what a call leaves in its workspace: the plan's tables (calls that reuse the plan, with
// whatever kernel, find them) and the status word.  They run beside the others and are done before them in batches of up to 128 requests and
// 8000 table entries (at the median, a call that plans takes no longer than one that reuses its plan); beyond, the call waits for them
// (193 .. 256 requests up to 8.7 us; more up to 18), and is still ahead of one with a plan kernel in front.
#include "seer_attention.h"
#include "seer_device.h"
#include "seer_plan_tables.h"
#include "seer_tile.h"

namespace seer {
namespace shortctx {

using namespace tile;

// Page ids outside the pool, among the entries that the requests' lengths reach: kBatch entries per thread and round, all of a
// round requested at once.
constexpr int kBatch = 8;
template <int THREADS>
struct TableCheck {
    int id[kBatch], n[kBatch], page[kBatch];
    __device__ __forceinline__ void request(const AttnArgs& a, int first) {
        const int entries = a.B * a.max_pages;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = min(first + k * THREADS + static_cast<int>(threadIdx.x), entries - 1);
            const int b = divide(i, a.max_pages, a.inv_pages);
            page[k] = i - b * a.max_pages;
            id[k] = a.block_table[i];
            n[k] = a.ctx_len[b];
        }
    }
    __device__ __forceinline__ bool outside(const AttnArgs& a) const {
        bool bad = false;
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            bad |= n[k] >= a.T && n[k] <= a.max_ctx && page[k] <= (n[k] - 1) / a.P && (id[k] < 0 || id[k] >= a.num_pages);
        return bad;
    }
};

}  // namespace shortctx

// TERMS: bf16 terms of a probability in the matrix product, as in the kernel that takes the shape's longer contexts.  NW waves, each with up
// to TILES tiles.
template <int DQK, int DV, int TERMS, int NW, int TILES>
__global__ __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(DQK > 128 && NW == 4 ? 1 : 2))) void attn_short_kernel(AttnArgs a, int extra) {
    using namespace shortctx;
    using S = Shape<DQK, DV>;
    constexpr int kThreads = NW * kWave, kChunks = DV / 4;              // 16-byte chunks of a row of sums
    static_assert(S::kStage >= 32 * DV * 4, "a wave's sums take the place of its tile");
    constexpr int kTiles = NW * S::kStage;
    static_assert(kTiles >= static_cast<int>(sizeof(PlanLds<kThreads>)), "");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kTiles];
    __shared__ float2 s_ml[NW][32];

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    if (static_cast<int>(blockIdx.x) < extra) {
        if (blockIdx.x == 0) {
            TableCheck<kThreads> check;
            check.request(a, 0);
            plan_tables<kThreads>(a, *reinterpret_cast<PlanLds<kThreads>*>(lds));
            bool bad = check.outside(a);
            for (int i = kBatch * kThreads; i < a.B * a.max_pages; i += kBatch * kThreads) {
                check.request(a, i);
                bad |= check.outside(a);
            }
            __syncthreads();                       // (the plan has set the status word)
            if (__any(bad) && lane == 0) atomicOr(&a.header->status, 2u);
        } else {
            plan_shared_pages(a, (blockIdx.x - 1) * kThreads, min(static_cast<int>(blockIdx.x) * kThreads, a.B), kThreads);
        }
        return;
    }
    // row blocks of 32 rows of one (request, KV head): on one XCD, so that all but the first find its tiles in that XCD's L2
    const int block = static_cast<int>(blockIdx.x) - extra;
    const int row_blocks = (a.G * a.T + 31) / 32;
    const int rest = block >> 3, rb = rest % row_blocks, item = rest / row_blocks * 8 + (block & 7);
    if (item >= a.B * a.Hkv) return;
    if (a.reuse_plan && !has_plan(a)) return;
    const int b = item / a.Hkv, kvh = item - b * a.Hkv;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ln = lane & 31, lg = lane >> 5;
    const int32_t* __restrict__ table = a.block_table + static_cast<size_t>(b) * a.max_pages;
    const unsigned char* __restrict__ kbase = static_cast<const unsigned char*>(a.k_pages);
    const unsigned char* __restrict__ vbase = static_cast<const unsigned char*>(a.v_pages);
    const bool page_pow2 = (a.P & (a.P - 1)) == 0;
    const int page_shift = __builtin_ctz(static_cast<unsigned>(a.P));
    auto page_of = [&](int tok) __attribute__((always_inline)) -> int { return page_pow2 ? tok >> page_shift : tok / a.P; };

    // ---- requested together: the length, the page ids of the tiles of this wave (tile i of it is tile wave + i * NW of the request; each
    //      lane the page of its own token, the lower lanes of even tiles, the upper ones of odd tiles), its query row and mask -------
    const int n = uniform_load(a.ctx_len + b);
    constexpr int kPairs = (TILES + 1) / 2;
    auto own_tok = [&](int j) __attribute__((always_inline)) -> int { return (wave + (TILES > 1 ? (2 * j + lg) * NW : 0)) * kTile + ln; };
    int row_of[kPairs];                            // page id, then row index in the pool, of this lane's token
#pragma unroll
    for (int j = 0; j < kPairs; ++j) row_of[j] = table[min(page_of(own_tok(j)), a.max_pages - 1)];
    const int r = rb * 32 + ln;
    const bool row_ok = r < a.G * a.T;
    const int t = row_ok ? r / a.G : 0;
    const int hq = kvh * a.G + (row_ok ? r - t * a.G : 0);
    uint64_t word = 0;
    if (row_ok) word = a.tree_mask ? a.tree_mask[static_cast<size_t>(b) * a.T + t] : (t >= 63 ? ~0ull : ((1ull << (t + 1)) - 1));
    if (a.T < 64) word &= (1ull << a.T) - 1;
    u32x4 qv[S::kKSteps];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.q) + ((static_cast<size_t>(b) * a.T + t) * a.Hq + hq) * DQK + lg * 8);
#pragma unroll
        for (int kk = 0; kk < S::kKSteps; ++kk) {
            qv[kk] = u32x4{0u, 0u, 0u, 0u};
            if (row_ok) qv[kk] = qp[kk * 2];
        }
    }
    const int n_tiles = tiles_of(n, a.T, a.max_ctx);      // none where the length cannot be used: zeros
    const int mine = wave < n_tiles ? (n_tiles - 1 - wave) / NW + 1 : 0;
    const int n0 = n - a.T;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        const int tok = own_tok(j), pg = min(max(row_of[j], 0), a.num_pages - 1);
        // (of 128 bytes or more each: 32 bits reach past the memory of the GPU)
        row_of[j] = static_cast<int>((static_cast<uint32_t>(pg) * a.Hkv + kvh) * static_cast<uint32_t>(a.P) + (tok - page_of(tok) * a.P));
    }
    // the row index in the pool of token `of` of this wave's tile i, for every lane
    auto pool_row = [&](int i, int of) __attribute__((always_inline)) -> uint32_t {
        int v = row_of[0];
#pragma unroll
        for (int j = 1; j < kPairs; ++j) {
            const int x = row_of[j];
            v = (i >> 1) == j ? x : v;
        }
        return __builtin_amdgcn_ds_bpermute((of + (TILES > 1 ? (i & 1) * 32 : 0)) << 2, v);
    };

    unsigned char* const stage = lds + wave * S::kStage;
    const int at = lds_addr(stage);
    constexpr int kKLoads = S::kKBytes / 1024, kVLoads = S::kVBytes / 1024;
    constexpr int kUnroll = DQK > 128 ? 4 : 8;     // (the wide heads have no registers for all loads' lane patterns)
    auto issue_k = [&](int i) __attribute__((always_inline)) {
        constexpr int kRow = S::kKRow / 16;
#pragma unroll kUnroll
        for (int j = 0; j < kKLoads; ++j) {
            const int c = j * kWave + lane, row = c / kRow, pos = c - row * kRow;
            const unsigned char* src = kbase + static_cast<size_t>(pool_row(i, row)) * S::kKRow + ((pos ^ k_swz<S::kKRow>(row)) << 4);
            __builtin_amdgcn_global_load_lds((const SEER_AS1 void*)(src), (SEER_AS3 void*)(stage + j * 1024), 16, 0, 0);
        }
    };
    auto issue_v = [&](int i) __attribute__((always_inline)) {
        constexpr int kRow = S::kVRow / 16;
#pragma unroll kUnroll
        for (int j = 0; j < kVLoads; ++j) {
            const int c = j * kWave + lane, row = c / kRow, pos = c - row * kRow;
            const unsigned char* src = vbase + static_cast<size_t>(pool_row(i, row)) * S::kVRow + ((pos ^ v_swz<S::kVRow>(row)) << 4);
            __builtin_amdgcn_global_load_lds((const SEER_AS1 void*)(src), (SEER_AS3 void*)(stage + S::kKBytes + j * 1024), 16, 0, 0);
        }
    };
    if (mine > 0) {
        issue_k(0);
        issue_v(0);
    }
    bf16x8 qreg[S::kKSteps];
#pragma unroll
    for (int kk = 0; kk < S::kKSteps; ++kk) {      // (the query rows are waited for here, not in the loop, where it would wait for tiles)
        asm volatile("" : "+v"(qv[kk]));
        qreg[kk] = as_bf16x8(qv[kk]);
    }
    {
        uint32_t lo = static_cast<uint32_t>(word), hi = static_cast<uint32_t>(word >> 32);
        asm volatile("" : "+v"(lo), "+v"(hi));
        word = (static_cast<uint64_t>(hi) << 32) | lo;
    }
    const Operands<DQK, DV> operands;
    f32x16 acc[S::kDTiles];
    float m_run = kNegInf, l_run = 0.f, top = kNegInf;
    // Three terms: a wave whose sums end up with an infinity or a NaN takes its tiles a second time, all of them scanned for V
    // rows that hold one (see the kernel of the longer contexts); otherwise only the tiles with masked slots are.
    for (int again = 0;; again = 1) {
#pragma unroll
        for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
        m_run = top = kNegInf, l_run = 0.f;
        if (again && mine > 0) {
            issue_k(0);
            issue_v(0);
        }
        for (int i = 0; i < mine; ++i) {
            const int tb = (wave + i * NW) * kTile, rel = tb - n0;      // uniform; a tile with masked slots has rel > -32
            const bool more = TILES > 1 && i + 1 < mine;
            wait_vmcnt<kVLoads>();                 // this tile's K rows (its V rows are behind them)
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s = tile_scores<DQK, DV>(at, operands, qreg);
            __builtin_amdgcn_sched_barrier(0);
            if (more) issue_k(i + 1);              // (the scores' reads of the stage have returned)
            if (rel > -kTile) tile_mask(s, word, rel);
            float alpha;
            uint32_t term[TERMS][8];
            tile_softmax<TERMS>(s, a.scale_log2, top, m_run, l_run, alpha, term);
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
                    for (int x = 0; x < 16; ++x) acc[dt][x] *= alpha;
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) wait_vmcnt<kKLoads>(); else wait_vmcnt<0>();
            __builtin_amdgcn_sched_barrier(0);
            // V rows past the end are cleared whatever they hold, rows with infinities or NaN to be added per row below
            const uint32_t past = tb + kTile > n ? ~0u << (n - tb) : 0u;
            uint32_t nonfinite = 0;
            if (TERMS > 1 ? rel > -kTile || again : past != 0) {
                unsigned char* const rows = stage + S::kKBytes;
                if constexpr (TERMS > 1) {
                    nonfinite = tile_nonfinite<DQK, DV>(rows, lane, kWave);
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) nonfinite |= __shfl_xor(nonfinite, o, kWave);
                    nonfinite = __builtin_amdgcn_readfirstlane(nonfinite) & ~past;
                }
                if (nonfinite | past) tile_clear_rows<DQK, DV>(rows, nonfinite | past, lane, kWave);
                __builtin_amdgcn_s_waitcnt(0xc07f);
                __builtin_amdgcn_sched_barrier(0);
            }
            tile_pv<DQK, DV, TERMS>(at, operands, term, acc);
            __builtin_amdgcn_sched_barrier(0);
            if (more) issue_v(i + 1);
            if constexpr (TERMS > 1)
                tile_add_rows<TERMS>(nonfinite, term, word, rel, acc, [&](int j) __attribute__((always_inline)) -> const uint16_t* {
                    return reinterpret_cast<const uint16_t*>(vbase) + static_cast<size_t>(pool_row(i, j)) * DV;
                });
        }
        if (TERMS == 1 || again) break;
        float sum0 = 0.f;                           // NaN iff some accumulator is infinite or NaN
#pragma unroll
        for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) sum0 = fmaf(acc[dt][i], 0.f, sum0);
        if (!__any(sum0 != 0.f)) break;
    }

    // ---- merge: every wave leaves its sums where its tiles were (16-byte chunk c of row r at c ^ r), then a thread adds eight columns of a
    //      row over the waves, in their order ---------------------------------------------------------------------------------------
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    if (mine > 0) {
        if (lg == 0) s_ml[wave][ln] = make_float2(m_run, l_tot);
        constexpr int kMask = (kChunks < 32 ? kChunks : 32) - 1;
#pragma unroll
        for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const int c = (dt * 8 + i4 * 2 + lg) ^ (ln & kMask);
                *reinterpret_cast<f32x4*>(stage + (ln * kChunks + c) * 16) = f32x4{acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
            }
    }
    __syncthreads();
    const int parts = min(NW, n_tiles);
    constexpr int kOct = DV / 8;
    for (int i = tid; i < 32 * kOct; i += kThreads) {
        const int row = i / kOct, oct = i - row * kOct, q_row = rb * 32 + row;
        if (q_row >= a.G * a.T) break;
        constexpr int kMask = (kChunks < 32 ? kChunks : 32) - 1;
        float M = kNegInf, L = 0.f, v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if (w < parts) M = fmaxf(M, s_ml[w][row].x);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (w >= parts) continue;
            const float2 ml = s_ml[w][row];
            const unsigned char* from = lds + w * S::kStage + row * kChunks * 16;
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(from + ((2 * oct) ^ (row & kMask)) * 16);
            const f32x4 x1 = *reinterpret_cast<const f32x4*>(from + ((2 * oct + 1) ^ (row & kMask)) * 16);
            // a wave that saw nothing for this row (m = -inf) may hold anything in its sums
            const bool live = ml.x != kNegInf;
            const float f = live ? fast_exp2(ml.x - M) : 0.f;
            L += live ? ml.y * f : 0.f;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                v[x] += live ? x0[x] * f : 0.f;
                v[4 + x] += live ? x1[x] * f : 0.f;
            }
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;           // a row that saw nothing: zeros
        u32x4 o;
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = pack_bf16x2(v[2 * x] * inv, v[2 * x + 1] * inv);
        const int q_t = q_row / a.G;
        *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(a.out) +
                                  ((static_cast<size_t>(b) * a.T + q_t) * a.Hq + kvh * a.G + (q_row - q_t * a.G)) * DV + oct * 8) = o;
    }
}

hipError_t launch_short(const AttnArgs& a, hipStream_t stream) {
    const int rows = a.G * a.T, row_blocks = (rows + 31) / 32;
    auto launch = [&](auto* kernel, int waves) {
        const int extra = a.reuse_plan ? 0 : 1 + (a.B + waves * kWave - 1) / (waves * kWave);
        const unsigned grid = static_cast<unsigned>((a.B * a.Hkv + 7) / 8) * 8u * row_blocks + extra;      // (short_workgroups())
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * kWave), 0, stream, a, extra);
        return hipGetLastError();
    };
    // (a second pair of tiles is looked up for longer tables only: heads of 128, tables of 8 and of 16 tiles 0.15 us less without it)
#define SEER_SHORT_CASE(DQK_, DV_, TERMS_, NW_, TILES_) \
    if (a.Dqk == DQK_ && a.Dv == DV_ && a.short_waves == NW_ && a.short_tiles <= NW_ * TILES_) return launch(&attn_short_kernel<DQK_, DV_, TERMS_, NW_, TILES_>, NW_);
    SEER_SHORT_CASE(128, 128, 1, 4, 1)
    SEER_SHORT_CASE(128, 128, 1, 8, 2)
    SEER_SHORT_CASE(128, 128, 1, 8, 3)
    SEER_SHORT_CASE(64, 64, 3, 4, 1)
    SEER_SHORT_CASE(64, 64, 3, 8, 2)
    SEER_SHORT_CASE(64, 64, 3, 8, 4)
    SEER_SHORT_CASE(256, 256, 3, 4, 1)
    SEER_SHORT_CASE(192, 128, 3, 4, 1)
    SEER_SHORT_CASE(192, 128, 3, 7, 2)
#undef SEER_SHORT_CASE
    return hipErrorInvalidValue;
}

}  // namespace seer
