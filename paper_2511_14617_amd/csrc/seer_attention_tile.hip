// Matrix-core verify-attention partition kernel for the head sizes beside D = 128: (64, 64), (256, 256) and
// (192, 128), separate K and V pools, pages of any size.
//
// What bounds it: HBM.  A KV token is read once for all R = G*T query rows of its head; with the scores and P.V on
// the matrix cores (64 MFMAs of 32 cycles per 32 KB tile and 32 rows at D = 256, 16 per 8 KB at D = 64) the
// arithmetic of a CU keeps up with more than its share of the bandwidth even though one wave runs a tile's phases one
// after the other, so the kernel leaves the overlap to the four to twelve waves of a CU instead of a hand-placed pipeline.
// The vector-ALU kernel it stands in for reads every KV token once per query row.  Measured, whole call: 16 requests, 16/4
// heads of 64, T = 9, 43 687 KV tokens 977 -> 31.9 us; 8/1 heads of 256, T = 5, same lengths 390 -> 39.9 us (with the plan
// and combine kernels as they are now).
//
// Work decomposition as in the D = 128 kernel: workgroup (stretch, KV head, row block), wave i owns query rows
// [32 i, 32 i + 32), the plan's stretches of 32-token tiles, one partial result per request touched.
// Data flow: a tile's K and V rows go HBM -> LDS directly, two stages; each lane picks the chunk its fixed LDS
// slot receives, so a tile may span any number of pages (the row index of every token comes from a 64-entry window of
// the block table by ds_bpermute).  S^T = K.Q^T, softmax with one query row per lane, O^T += V^T.P^T.
//
// Precision: the vector-ALU kernel multiplies fp32 probabilities into V.  A probability goes into the bf16 matrix
// product as three terms, its bf16 rounding and twice the bf16 rounding of what is left, which hold all its 24 bits,
// and the row sums take the fp32 value, so the output differs from the vector kernel's by the order of the fp32 sums
// only (two terms, good to 16 bits, would save 3 %: 31.9 -> 30.8 and 39.9 -> 39.4 us).  V rows that hold infinities or NaN in a tile with masked slots are kept out of the product
// (0 * NaN must not reach rows that do not see the slot) and added per row.
#include <type_traits>

#include "seer_attention.h"
#include "seer_device.h"
#include "seer_plan.h"
#include "seer_tile.h"

namespace seer {

// One wave per 32 query rows.  Registers: 64-wide heads leave room for three waves per SIMD, (192, 128) for two; at D = 256
// Q^T and O^T alone take 192, so one wave has a SIMD to itself (with 256 registers 40 of them would be spilled, and a
// spill's reload waits for the tile loads in flight).
// SELF: every wave finds its stretch itself (seer_plan.h) instead of reading it from the plan kernel's tables.
template <int DQK, int DV, bool SELF>
__global__ __launch_bounds__(tile_max_waves(DQK) * kWave) __attribute__((amdgpu_waves_per_eu(tile_waves_per_simd(DQK))))
void attn_tile_kernel(AttnArgs a, int n_waves) {
    using namespace tile;
    using S = Shape<DQK, DV>;
    static_assert(S::kStage == tile_stage_kb(DQK, DV) * 1024 && kTile == kPlanTile, "the host sizes the launch with the same numbers");
    // two stages of K tile, V tile; then two words: the scanned tile's tokens with infinities or NaN, "take the piece again"
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * S::kStage + 16];
    __shared__ int s_line[kLineWords];              // (see plan_stretch)
    volatile uint32_t* s_nonfinite = reinterpret_cast<volatile uint32_t*>(lds + 2 * S::kStage);
    volatile uint32_t* s_again = s_nonfinite + 1;

    int rest = blockIdx.x >> 3;                     // (the grid's layout: see the D = 128 kernel)
    const int kvh = rest % a.Hkv;
    rest /= a.Hkv;
    const int rb = rest % a.row_blocks;
    const int wg = (rest / a.row_blocks) * 8 + (blockIdx.x & 7);
    if (wg >= a.wgs_per_head) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ln = lane & 31, lg = lane >> 5;

    StretchRec rec;
    bool new_history = false;
    if (SELF) {
        const SelfPlan own = plan_stretch(a, s_line, wg);
        rec = own.rec, new_history = own.new_history;
        if (rec.b < 0) {
            publish_stretch(a, s_line, rec, wg, kvh, rb, wave, false);
            if (new_history && tid == 0) record_speed(a, wg, kvh, rb, 0, 0, true);
            return;
        }
    } else {
        rec = uniform_stretch(a, wg);
    }
    int b = rec.b;
    if (b < 0) return;
    const int slot_bias = a.balanced ? wg : 0;
    int g = rec.tile_begin;
    const int g_end = rec.tile_end;
    const int g_first = g;
    const uint64_t clock_begin = __builtin_amdgcn_s_memrealtime();
    bool bad_page = false;

    const unsigned char* __restrict__ kbase = static_cast<const unsigned char*>(a.k_pages);
    const unsigned char* __restrict__ vbase = static_cast<const unsigned char*>(a.v_pages);
    const int lds0 = lds_addr(lds);
    const bool page_pow2 = (a.P & (a.P - 1)) == 0;
    const int page_shift = __builtin_ctz(static_cast<unsigned>(a.P));
    auto page_of = [&](int tok) __attribute__((always_inline)) -> int { return page_pow2 ? tok >> page_shift : tok / a.P; };

    const Operands<DQK, DV> operands;

    // A piece's start needs the request's first and last tile and its length (lanes 0, 1, 2 of `words`) and its first window of
    // page ids.  They are requested together, for the first piece right behind the stretch's record and for each further
    // one while the piece before it is worked on: loaded where they are used they were three round trips more per piece (whole call,
    // 16 requests, heads of 64: 33.2 -> 32.0 us, of 192/128: 45.5 -> 44.0, of 256: 39.7 -> 39.5).
    int words = 0, pages = 0;
    auto request = [&](int req, int first_page) __attribute__((always_inline)) {
        req = min(req, a.B - 1);
        if (!SELF) words = *(lane < 2 ? a.tile_off + req + lane : a.ctx_len + req);
        pages = a.block_table[static_cast<size_t>(req) * a.max_pages + min(first_page + lane, a.max_pages - 1)];
    };
    request(b, page_of((g - rec.req_begin) * kTile));

  for (; g < g_end; ++b) {
    if (SELF) words = line_words(s_line, b);
    const int t_lo = __builtin_amdgcn_readlane(words, 0), t_hi = __builtin_amdgcn_readlane(words, 1);
    if (t_hi == t_lo) {
        request(b + 1, 0);
        continue;
    }
    const int item_idx = b + slot_bias;
    const int n = __builtin_amdgcn_readlane(words, 2);
    const int tok_begin = (g - t_lo) * kTile;
    const int tok_end = min(n, (min(g_end, t_hi) - t_lo) * kTile);
    g = t_hi;
    const int n0 = n - a.T;
    const int n_tiles = (tok_end - tok_begin + kTile - 1) / kTile;
    bare_barrier();                                // every wave is done with the previous piece's stages
    if (tid == 0) *s_again = 0;

    // ---- page window and tile loads ---------------------------------------------------------
    const int32_t* __restrict__ table = a.block_table + static_cast<size_t>(b) * a.max_pages;
    const int last_page = (n - 1) / a.P;
    int win = 0, pg_win = 0;                       // lane l holds the (clamped) page id of logical page win + l
    auto set_window = [&](int first, int pg) __attribute__((always_inline)) {
        win = first;
        if (pg < 0 || pg >= a.num_pages) {
            if (first + lane <= last_page) bad_page = true;
            pg = min(max(pg, 0), a.num_pages - 1);
        }
        pg_win = pg;
    };
    set_window(page_of(tok_begin), pages);
    auto issue_tile = [&](int tile, int stage) __attribute__((always_inline)) {
        const int tb = tok_begin + tile * kTile;
        const int first = page_of(tb);
        if (first < win || page_of(tb + kTile - 1) >= win + kWave)            // uniform; a tile spans at most 32 pages
            set_window(first, table[min(first + lane, a.max_pages - 1)]);
        const int tok = tb + ln, lp = page_of(tok);
        const int pg = __builtin_amdgcn_ds_bpermute((lp - win) << 2, pg_win);
        // row index in the pool (of 128 bytes or more each: 32 bits reach past the memory of the GPU)
        const uint32_t row_idx = (static_cast<uint32_t>(pg) * a.Hkv + kvh) * static_cast<uint32_t>(a.P) + (tok - lp * a.P);
        constexpr int kKChunks = S::kKRow / 16, kVChunks = S::kVRow / 16;
        for (int j = wave; j < S::kKBytes / 1024; j += n_waves) {
            const int c = j * kWave + lane, row = c / kKChunks, pos = c - row * kKChunks;
            const uint32_t r = __builtin_amdgcn_ds_bpermute(row << 2, row_idx);
            const unsigned char* src = kbase + static_cast<size_t>(r) * S::kKRow + ((pos ^ k_swz<S::kKRow>(row)) << 4);
            __builtin_amdgcn_global_load_lds((const SEER_AS1 void*)(src), (SEER_AS3 void*)(lds + stage + j * 1024), 16, 0, 2);
        }
        for (int j = wave; j < S::kVBytes / 1024; j += n_waves) {
            const int c = j * kWave + lane, row = c / kVChunks, pos = c - row * kVChunks;
            const uint32_t r = __builtin_amdgcn_ds_bpermute(row << 2, row_idx);
            const unsigned char* src = vbase + static_cast<size_t>(r) * S::kVRow + ((pos ^ v_swz<S::kVRow>(row)) << 4);
            __builtin_amdgcn_global_load_lds((const SEER_AS1 void*)(src), (SEER_AS3 void*)(lds + stage + S::kKBytes + j * 1024), 16, 0, 2);
        }
    };

    // ---- this lane's query row ---------------------------------------------------------------
    const int r = rb * a.rows_per_block + wave * 32 + ln;
    const bool row_ok = r < min(a.G * a.T, (rb + 1) * a.rows_per_block);
    const int t = row_ok ? r / a.G : 0;
    const int hq = kvh * a.G + (row_ok ? r - t * a.G : 0);
    uint64_t word = 0;
    if (row_ok) word = a.tree_mask ? a.tree_mask[static_cast<size_t>(b) * a.T + t] : (t >= 63 ? ~0ull : ((1ull << (t + 1)) - 1));
    if (a.T < 64) word &= (1ull << a.T) - 1;
    bf16x8 qreg[S::kKSteps];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(
            static_cast<const uint16_t*>(a.q) + ((static_cast<size_t>(b) * a.T + t) * a.Hq + hq) * DQK + lg * 8);
#pragma unroll
        for (int kk = 0; kk < S::kKSteps; ++kk) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (row_ok) v = qp[kk * 2];
            qreg[kk] = as_bf16x8(v);
        }
    }
    if (g < g_end) request(b + 1, 0);
    // A piece whose accumulators end up with an infinity or a NaN is taken a second time with every tile scanned for V
    // rows that hold one (see the head of the file); otherwise only the tiles with masked slots are.
    f32x16 acc[S::kDTiles];
    float m_run, l_run;
    for (int scan_all = 0;; scan_all = 1) {
    issue_tile(0, 0);
#pragma unroll
    for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    m_run = kNegInf, l_run = 0.f;

    for (int u = 0; u < n_tiles; ++u) {
        const int stage = (u & 1) * S::kStage;
        wait_vmcnt<0>();
        bare_barrier();                            // tile u has landed for every wave, every wave is done with tile u - 1
        if (u + 1 < n_tiles) issue_tile(u + 1, S::kStage - stage);
        __builtin_amdgcn_sched_barrier(0);
        const int tb = tok_begin + u * kTile;
        const int rel = tb - n0;                    // uniform; a tile with masked slots has rel > -32
        uint32_t nonfinite = 0;                    // uniform: tokens of this tile whose V row is kept out of the product
        if (rel > -kTile || scan_all) {
            // V rows past the end of the request are cleared whatever they hold; rows with infinities or NaN are cleared
            // too and added per row below.
            unsigned char* vl = lds + stage + S::kKBytes;
            if (tid == 0) *s_nonfinite = 0;
            __builtin_amdgcn_s_waitcnt(0xc07f);
            bare_barrier();
            uint32_t found = tile_nonfinite<DQK, DV>(vl, tid, n_waves * kWave);
            if (tb + kTile > n) found &= (1u << (n - tb)) - 1;
            if (found) atomicOr(const_cast<uint32_t*>(s_nonfinite), found);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            bare_barrier();
            nonfinite = __builtin_amdgcn_readfirstlane(*s_nonfinite);
            const uint32_t cleared = nonfinite | (tb + kTile > n ? ~((1u << (n - tb)) - 1) : 0u);
            if (cleared) {
                tile_clear_rows<DQK, DV>(vl, cleared, tid, n_waves * kWave);
                __builtin_amdgcn_s_waitcnt(0xc07f);
            }
            bare_barrier();
        }

        // ---- scores, softmax with one query row per lane, O^T += V^T . P^T --------------------------------
        f32x16 s = tile_scores<DQK, DV>(lds0 + stage, operands, qreg);
        if (rel > -kTile) tile_mask(s, word, rel);
        float alpha;
        uint32_t term[3][8];
        tile_softmax<3>(s, a.scale_log2, m_run, m_run, l_run, alpha, term);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
        }
        tile_pv<DQK, DV, 3>(lds0 + stage, operands, term, acc);
        tile_add_rows<3>(nonfinite, term, word, rel, acc, [&](int j) __attribute__((always_inline)) -> const uint16_t* {
            const int tok = tb + j, lp = page_of(tok);
            const int pg = min(max(table[min(lp, a.max_pages - 1)], 0), a.num_pages - 1);
            return reinterpret_cast<const uint16_t*>(vbase) + ((static_cast<size_t>(pg) * a.Hkv + kvh) * a.P + (tok - lp * a.P)) * DV;
        });
    }

    float sum0 = 0.f;                               // NaN iff some accumulator is infinite or NaN
#pragma unroll
    for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) sum0 = fmaf(acc[dt][i], 0.f, sum0);
    if (scan_all) break;
    if (__any(sum0 != 0.f) && lane == 0) *s_again = 1;
    __builtin_amdgcn_s_waitcnt(0xc07f);
    bare_barrier();                                // (also: every wave is done with the stages)
    if (!__builtin_amdgcn_readfirstlane(*s_again)) break;
    }

    // ---- partial result: (reference exponent, sum, unnormalised O) per row ---------------------
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    if (row_ok) {
        const size_t prow = (static_cast<size_t>(item_idx) * a.T + t) * a.Hq + hq;
        if (lg == 0) {
            a.part_ml[2 * prow] = m_run;
            a.part_ml[2 * prow + 1] = l_tot;
        }
        float* __restrict__ po = a.part_acc + prow * DV + lg * 4;
#pragma unroll
        for (int dt = 0; dt < S::kDTiles; ++dt)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4)
                *reinterpret_cast<f32x4*>(po + dt * 32 + i4 * 8) =
                    f32x4{acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
    }
  }  // pieces of the stretch
    if constexpr (SELF) publish_stretch(a, s_line, rec, wg, kvh, rb, wave, bad_page);
    else if (__any(bad_page) && lane == 0) atomicOr(&a.header->status, 2u);
    // speed history for the next call's plan (see the D = 128 kernel)
    if (a.balanced && !a.fixed_split && tid == 0)
        record_speed(a, wg, kvh, rb, __builtin_amdgcn_s_memrealtime() - clock_begin, g_end - g_first, new_history);
}

hipError_t launch_tile(const AttnArgs& a, hipStream_t stream) {
    const int nw = a.rows_per_block / 32;
    const dim3 grid(static_cast<unsigned>((a.wgs_per_head + 7) / 8) * 8u * static_cast<unsigned>(a.Hkv) *
                    static_cast<unsigned>(a.row_blocks));
#define SEER_TILE_CASE(DQK_, DV_)                                                                                      \
    if (a.Dqk == DQK_ && a.Dv == DV_) {                                                                                \
        if (a.self_plan) hipLaunchKernelGGL((attn_tile_kernel<DQK_, DV_, true>), grid, dim3(nw * kWave), 0, stream, a, nw);      \
        else hipLaunchKernelGGL((attn_tile_kernel<DQK_, DV_, false>), grid, dim3(nw * kWave), 0, stream, a, nw);                 \
        return hipGetLastError();                                                                                      \
    }
    SEER_TILE_CASE(64, 64)
    SEER_TILE_CASE(256, 256)
    SEER_TILE_CASE(192, 128)
#undef SEER_TILE_CASE
    return hipErrorInvalidValue;
}

}  // namespace seer
