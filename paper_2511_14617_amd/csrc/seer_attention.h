// Internal declarations shared by the verify-attention sources: the split-K
// plan that lives at the head of the caller's workspace, and the launchers of
// the individual kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/seer_verify.h"

namespace seer {

// Split-K work is planned ON THE DEVICE from ctx_len (the host never sees the
// lengths, so it cannot size partitions without a synchronisation).
//
// Balanced ("stream") partitioning: per KV head, the 32-token tiles of all
// requests are laid end to end, request after request, and that line is cut
// into W stretches, one per workgroup.  W x Hkv is chosen to be what the GPU
// holds at once, so there is a single round of workgroups and every one of
// them streams about the same number of KV bytes, whatever the mix of lengths
// -- eight 100k-token stragglers and several hundred short requests both fill
// all 256 CUs.  A stretch that crosses a request boundary yields one partial
// result per request it touches.  The piece of request b in stretch w has partial slot w + b: along
// the line every next piece raises w, b or both, so slots are unique and below W + B, and nobody
// has to count pieces.  Request b owns consecutive slots, which the combine kernel merges.
//
// Stretch lengths follow the measured speed of each workgroup slot.  Workgroups
// that stream the same number of bytes do not finish together: on this part the
// eight XCDs differ by about 12 % in sustained gather bandwidth, and of two
// workgroups resident on one CU the one dispatched first is served first.  Both
// are properties of the workgroup's index (the grid is laid out so that the
// workgroups with the same stretch index w, one per KV head, share XCD and
// dispatch round), and stable from call to call.  So every partition workgroup
// adds its tiles and its duration (constant 100 MHz clock) to two counters of
// its stretch index in the workspace (where a call that plans for itself finds no history, and nothing has cleared counters, one
// workgroup of a stretch index sets them), and the next call's plan cuts the line in
// proportion to the smoothed tiles-per-time of each index (clamped to
// [3/4, 4/3] of the mean).  The sums of these rates that a cut needs are made at the end of a call that plans,
// by a workgroup of the combine kernel.  The history lies at one place and has one size in every layout, so that no
// other part of a workspace ever comes to lie there and it outlives a change of the batch.  A workspace that holds no
// valid history (first use, other W, sums that no rates can have: share_ok in seer_plan.h) gives equal stretches;
// SEER_ATTN_FIXED_SPLIT always does.
struct PlanHeader {
    uint32_t status;     // bit 0: bad ctx_len somewhere; bit 1: page id out of range
    int32_t plan_b, plan_w;  // the batch and the split the tables are for (see plan_b_word, plan_w_word)
    uint32_t fb_magic;     // kFeedbackMagic once the speed history below the header is meaningful
    int32_t fb_w;          // W it was recorded for
};
constexpr uint32_t kFeedbackMagic = 0x5ee2fb01u;
constexpr int kMaxWgsPerHead = 1024;   // 256 CUs x 4 resident workgroups, one KV head
constexpr int kHistoryStride = kMaxWgsPerHead + 4;     // words from one array of the history to the next (16-byte loads of five words)

// A call that reuses a plan reads tables that it did not write itself.  They index by request and by stretch and nothing else
// steers an unchecked access, so tables made for the same number of requests and the same stretches keep every access in
// bounds whatever else differs; the kernels compare these two words of the header first and do nothing if they differ.
__host__ __device__ inline int32_t plan_b_word(int B) { return B ^ 0x2d35c0de; }
__host__ __device__ inline int32_t plan_w_word(int W, bool balanced) { return balanced ? W : -W; }

// A stretch as its workgroups need it, in one 16-byte load: the request in which it starts (-1: nothing to do), its tiles
// on the line, and that request's first tile (with it the first page ids can be requested beside the request's other words
// instead of behind them).
struct StretchRec {
    int32_t b, tile_begin, tile_end, req_begin;
};

// The partial slots of a request, first .. last (none: last < first).
struct ReqSlots {
    int32_t first, last;
};

// Up to this many requests the tiled kernels plan for themselves (seer_plan.h):
// one per lane of a wave.  Whole call with the plan kernel | without: 4 requests of 64 .. 512 tokens 16.9 | 14.1 us, 16 requests with heads of
// 64 31.9 | 27.6, of 256 40.0 | 36.0, 64 requests on one KV head 57.1 | 53.5, on eight 237.3 | 233.3; shared
// latent, two requests, 33.7 | 30.0.  (0.2 .. 0.5 us of the second figures is the look at the whole history, share_ok.)  (Not all of the plan kernel's 5.5 us:
// the partition kernel begins 1.8 us later, most of it the fetch of the additional code.)
constexpr int kSelfPlanRequests = 64;

constexpr int kPlanTile = 32;          // tokens per scheduling tile
// Tiles of a stretch, at least, where the batch is too short for the chip: one tile where a workgroup's time is the chain of its
// tiles (whole call, 4 requests of 64 .. 512 tokens: 22.7 us with four tiles, 21.1 with two, 17.9 with one; 2 requests of
// 64 .. 600 with heads of 64: 21.5, 18.6, 17.7; batches that fill the chip do not change).  The shapes of the shared-latent kernel, whose
// pieces leave partial results of 256 KB per row block, and of the general kernel keep four (2 requests of 1000 .. 4000 tokens: 56.2 us
// with four, 58.4 with one).  D = 128 keeps four as well once every stretch has two or three tiles anyway and the pieces would leave more
// than kFinePartialsBelow: the shorter chain then saves less than the additional pieces cost in stores and in the combine kernel (75
// requests of 150 tokens, 16/2 heads, 16 slots, 33 MB: 33.5 us with two tiles, 29.8 with four; 162, 8/2, 40 MB: 38.5, 38.1; but 144, 2/1, 10
// slots, 10 MB: 28.1, 31.1; 3 of 10 000 .. 20 000, 8/1, 9 slots, 19 MB: 27.7, 28.9).
constexpr size_t kFinePartialsBelow = size_t{24} << 20;
constexpr int kMinTilesLatent = 4, kMinTiles = 1;
// Stretches follow the measured speeds only from here on (tiles per stretch): below, rounding to tiles decides.
constexpr int kMinTilesWeighted = 8;
constexpr int kDefaultMaxSplits = 256;
constexpr int kNumCU = 256;            // MI355X

struct WorkspaceLayout {
    int max_items;
    int wgs_per_head;    // W (balanced mode) or B (one workgroup per request)
    int max_splits;
    int row_blocks;
    size_t off_header, off_fb, off_slots, off_tiles, off_stretch, off_shared, off_flags, off_ml, off_acc, total;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Ring depth D of the tiled GQA kernel (tiles in flight per workgroup while one is computed;
// the K ring and the V ring have D + 1 slots of 8 KB each), by waves per workgroup.  Two-wave
// workgroups run four to a CU and keep one tile in flight each; larger ones run at most two to a CU.
// Measured on the 8B- to 72B-class shapes: between depths 1 and 4 the time changes by a few per cent only.
constexpr int gqa_pipe_depth(int waves) { return waves <= 2 ? 1 : 3; }

// Partial results of the tiled D = 128 kernel are written with non-temporal stores while all of them are
// small: measured on the 8B-class shapes, the partition kernel of the grouped-rollout batch (28 MB of
// partials) is 2.7 % faster with them and the call 2 %, the long-tail batch (20 MB) does not care, and the
// multi-path batch (86 MB) loses 1 % of the call, because the combine kernel then fetches from DRAM what it
// would otherwise find in the memory-side cache.
constexpr size_t kStreamPartialsBelow = size_t{64} << 20;

// The tiled D = 128 kernel handles up to 256 query rows (8 waves) of a KV head per workgroup; a request
// with more rows per KV head (large groups of heads times a wide draft tree) is cut into row blocks of
// equal size, each a workgroup of its own walking the same stretch (placed on the same XCD, so all but
// the first find the tiles in that XCD's L2).
inline bool gqa_page_size_ok(int P) { return P >= 16 && P <= 1024 && (P & (P - 1)) == 0; }
inline int gqa_row_blocks(int rows) { return (rows + 255) / 256; }
// A row block of 129 .. 144 rows is served, where pieces are long, by two sets of four waves on alternate tiles, four of which
// share the leftover rows (see the kernel), instead of by a fifth wave; such a block keeps its exact row count.
inline bool gqa_block_uses_helpers(int rows_per_block) { return rows_per_block > 128 && rows_per_block <= 144; }
inline int gqa_rows_per_block(int rows) {
    const int nb = gqa_row_blocks(rows);
    const int per = (rows + nb - 1) / nb;
    return gqa_block_uses_helpers(per) ? per : (per + 31) / 32 * 32;
}
inline int gqa_waves_per_block(int rows_per_block) { return gqa_block_uses_helpers(rows_per_block) ? 8 : rows_per_block / 32; }

// The tiled kernel for the other head sizes (seer_attention_tile.hip): any page size, separate K and V pools, two LDS stages
// of one K and one V tile, row blocks of as many waves as a workgroup holds.
inline bool tile_shape(int Dqk, int Dv) { return (Dqk == 64 && Dv == 64) || (Dqk == 256 && Dv == 256) || (Dqk == 192 && Dv == 128); }
// Every workspace is laid out, and every plan made, by the shape alone, also for calls that force the general kernel (it
// walks whatever stretches it finds): a plan is reused by calls whose flags differ.
inline bool tile_layout(const seer_attn_params& p) { return tile_shape(p.Dqk, p.Dv) && !p.kv_shared_latent; }
inline bool gqa_layout(const seer_attn_params& p) { return p.Dqk == 128 && p.Dv == 128 && gqa_page_size_ok(p.page_size) && !p.kv_shared_latent; }
inline bool mla_layout(const seer_attn_params& p) {
    return p.Dqk == 576 && p.Dv == 512 && p.page_size >= 32 && gqa_page_size_ok(p.page_size) && p.kv_shared_latent;
}
inline bool tile_supports(const seer_attn_params& p) { return tile_layout(p) && !(p.flags & SEER_ATTN_GENERAL_KERNEL); }
// (also a matter of the shape alone; calls that force the general kernel or reuse a plan do not use it)
inline bool self_plan_layout(const seer_attn_params& p) {
    return p.B <= kSelfPlanRequests && p.max_splits != 1 && (gqa_layout(p) || tile_layout(p) || mla_layout(p));
}
constexpr int tile_stage_kb(int Dqk, int Dv) { return 32 * 2 * (Dqk + Dv) / 1024; }
constexpr int tile_waves_per_simd(int Dqk) { return Dqk == 64 ? 3 : (Dqk == 256 ? 1 : 2); }
constexpr int tile_max_waves(int Dqk) { return Dqk == 256 ? 4 : 8; }     // per workgroup
inline int tile_row_blocks(int rows, int Dqk) { return (rows + tile_max_waves(Dqk) * 32 - 1) / (tile_max_waves(Dqk) * 32); }
inline int tile_rows_per_block(int rows, int Dqk) {
    const int nb = tile_row_blocks(rows, Dqk);
    return ((rows + nb - 1) / nb + 31) / 32 * 32;
}

// Requests taken whole, one workgroup per 32 query rows of a KV head (seer_attention_short.hip): the waves of such a workgroup by the tiles
// that a table has for them, and whether a call is one.  The block table's width is what the host knows of the lengths.
inline int short_waves(int Dqk, int tiles) { return Dqk == 256 || tiles <= 4 ? 4 : (Dqk == 192 ? 7 : 8); }
constexpr int kShortTableEntries = 16384;      // page ids that one workgroup looks through for the status word
inline int short_tiles(const seer_attn_params& p) {
    const long long t = (static_cast<long long>(p.max_pages_per_seq) * p.page_size + 31) / 32;
    return t > 1 << 20 ? 1 << 20 : static_cast<int>(t);
}
inline long long short_workgroups(const seer_attn_params& p) {      // (groups of eight items, one to each XCD)
    return (static_cast<long long>(p.B) * p.Hkv + 7) / 8 * 8 * (((p.Hq / p.Hkv) * p.T + 31) / 32);
}
bool short_call(const seer_attn_params& p);

// Workgroups of the partition kernel that one CU holds at once, by kernel shape.
inline int resident_wgs_per_cu(const seer_attn_params& p) {
    if (tile_layout(p)) {
        const int waves = tile_rows_per_block((p.Hq / p.Hkv) * p.T, p.Dqk) / 32;
        const int by_waves = 4 * tile_waves_per_simd(p.Dqk) / waves;
        const int by_lds = 159 / (2 * tile_stage_kb(p.Dqk, p.Dv) + 1);
        const int n = by_waves < by_lds ? by_waves : by_lds;
        return n < 1 ? 1 : (n > 8 ? 8 : n);
    }
    if (!gqa_layout(p)) return 4;
    const int waves = gqa_waves_per_block(gqa_rows_per_block((p.Hq / p.Hkv) * p.T));   // one wave per 32 query rows
    const int by_waves = 8 / waves;                       // 2 waves per SIMD, 4 SIMDs
    const int depth = gqa_pipe_depth(waves);
    // 160 KB of LDS per CU, 16 KB per ring slot pair; five 32 KB workgroups would need all of it and
    // do not become resident together (measured: a fifth of the grid ran as a second round)
    const int by_lds = 159 / (16 * (depth + 1));
    return by_waves < 1 ? 1 : (by_waves < by_lds ? by_waves : by_lds);
}

// Host-only arithmetic; the plan kernel is given the same numbers.
inline WorkspaceLayout workspace_layout(const seer_attn_params& p) {
    WorkspaceLayout w{};
    w.max_splits = p.max_splits > 0 ? p.max_splits : kDefaultMaxSplits;
    const int rows_per_head = (p.Hq / p.Hkv) * p.T;
    w.row_blocks = gqa_layout(p) ? gqa_row_blocks(rows_per_head) : 1;
    if (mla_layout(p)) w.row_blocks = (rows_per_head + 127) / 128;
    else if (tile_layout(p)) w.row_blocks = tile_row_blocks(rows_per_head, p.Dqk);
    if (w.max_splits == 1) {
        w.wgs_per_head = p.B;
        w.max_items = p.B;
    } else {
        if (mla_layout(p)) {
            // one 4-wave workgroup per CU; a request's rows are cut into blocks of 128, and the
            // row-block workgroups of one stretch are launched as a group on one XCD (groups of 8 stretches)
            w.wgs_per_head = 8 * (kNumCU / (8 * w.row_blocks * p.Hkv));
            if (w.wgs_per_head < 1) w.wgs_per_head = kNumCU / (w.row_blocks * p.Hkv);
        } else {
            w.wgs_per_head = kNumCU * resident_wgs_per_cu(p) / (p.Hkv * w.row_blocks);
            if (w.wgs_per_head > kMaxWgsPerHead) w.wgs_per_head = kMaxWgsPerHead;
        }
        if (w.wgs_per_head < 1) w.wgs_per_head = 1;
        // a stretch adds one piece per request boundary it crosses: pieces <= W + B
        w.max_items = w.wgs_per_head + p.B;
    }
    const size_t rows = static_cast<size_t>(w.max_items) * p.T * p.Hq;
    const size_t per_b = sizeof(int32_t) * (static_cast<size_t>(p.B) + 1);
    w.off_header = 0;
    w.off_fb = 256;                    // time[W], tiles[W], smoothed speed[W], shares of the rates[W], whatever the shape
    w.off_slots = align_up(w.off_fb + 4 * sizeof(uint32_t) * kHistoryStride, 256);
    w.off_tiles = align_up(w.off_slots + sizeof(ReqSlots) * p.B, 256);
    w.off_stretch = align_up(w.off_tiles + per_b, 256);
    w.off_shared = align_up(w.off_stretch + sizeof(StretchRec) * w.wgs_per_head, 256);
    w.off_flags = align_up(w.off_shared + per_b, 256);            // one byte per wave of the partition kernel's grid
    const bool self_plans = self_plan_layout(p);
    w.off_ml = align_up(w.off_flags + (self_plans ? size_t{8} * w.wgs_per_head * p.Hkv * w.row_blocks : 0), 256);
    w.off_acc = align_up(w.off_ml + 2 * sizeof(float) * rows, 256);
    w.total = align_up(w.off_acc + sizeof(float) * rows * p.Dv, 256);
    return w;
}

// floor(2^32 / d), or the largest number below 2^32 (see divide() in seer_plan.h).
inline uint32_t reciprocal(uint32_t d) { return d > 1 ? static_cast<uint32_t>((uint64_t{1} << 32) / d) : 0xffffffffu; }

// Everything a kernel needs, by value.
struct AttnArgs {
    void* out;
    const void* q;
    const void* k_pages;
    const void* v_pages;     // nullptr: shared latent
    const int32_t* block_table;
    const int32_t* ctx_len;
    const uint64_t* tree_mask;
    PlanHeader* header;
    const ReqSlots* req_slots;      // [B]
    const int32_t* tile_off;        // [B+1] first tile of each request on the per-head tile line
    const StretchRec* stretch;      // [wgs_per_head]
    const int32_t* shared_tiles;  // [B] leading tiles of each request whose pages a neighbouring request maps too
    uint32_t* fb_time;          // [wgs_per_head] sum over KV heads of the workgroup's duration, 10 ns ticks
    uint32_t* fb_tiles;         // [wgs_per_head] sum over KV heads of the tiles it streamed
    float* fb_speed;            // [wgs_per_head] smoothed tiles per tick
    uint32_t* fb_before;        // [wgs_per_head] share of the rates in front of a stretch index, in units of 2^-32
    uint8_t* page_flags;        // [wgs_per_head][Hkv][row_blocks][8] see publish_stretch
    int32_t self_plan;          // 1: the partition kernel plans for itself
    int32_t plan_waves;         // waves of a workgroup of the partition kernel
    int32_t reuse_plan;         // 1: the tables of an earlier call
    int32_t max_splits, max_ctx;   // most pieces of a request; most tokens that a row of the block table holds
    uint32_t inv_wgs, inv_splits;   // reciprocal() of wgs_per_head and of max_splits - 1
    int32_t fixed_split;        // 1: equal stretches, no history read or written (also where there is one stretch only)
    int32_t balanced;           // 0: one workgroup per request (max_splits == 1), slot = request, no history either
    int32_t min_tiles;          // tiles of a stretch, at least (see kMinTiles)
    int32_t fine_pieces;        // with more pieces than this in stretches of two or three tiles: four tiles (see kFinePartialsBelow)
    int32_t short_waves, short_tiles;   // requests taken whole: waves of a workgroup, tiles of the table
    uint32_t inv_pages;         // reciprocal() of max_pages
    int32_t stream_only;        // 1: the tiled D = 128 kernel only streams its tiles (diagnostic)
    int32_t stream_partials;    // 1: the tiled D = 128 kernel writes its partial results with non-temporal stores
    int32_t row_blocks, rows_per_block;   // tiled kernels: workgroups per (stretch, KV head); rows of each (D = 128 and the other head sizes)
    float* part_ml;             // [max_items][T][Hq][2]  (running max in log2 units, sum)
    float* part_acc;            // [max_items][T][Hq][Dv] unnormalised
    int32_t B, T, Hq, Hkv, G, Dqk, Dv, P, num_pages, max_pages, wgs_per_head;
    float scale_log2;           // scale * log2(e): scores are kept in base-2 units
};

// Does the workspace hold a plan for this call's batch and split?
__device__ __forceinline__ bool has_plan(const AttnArgs& a) {
    const int32_t b = a.header->plan_b, w = a.header->plan_w;
    return __builtin_amdgcn_readfirstlane(b) == plan_b_word(a.B) &&
           __builtin_amdgcn_readfirstlane(w) == plan_w_word(a.wgs_per_head, a.balanced != 0);
}

// The record of stretch wg, moved to scalar registers (one load, requested together with the header's words; see uniform_load);
// nothing to do where there is no plan.
__device__ __forceinline__ StretchRec uniform_stretch(const AttnArgs& a, int wg) {
    const int4 v = *reinterpret_cast<const int4*>(a.stretch + wg);
    const bool planned = has_plan(a);
    return {planned ? __builtin_amdgcn_readfirstlane(v.x) : -1, __builtin_amdgcn_readfirstlane(v.y), __builtin_amdgcn_readfirstlane(v.z),
            __builtin_amdgcn_readfirstlane(v.w)};
}

hipError_t launch_plan(const AttnArgs& a, hipStream_t stream);
hipError_t launch_general(const AttnArgs& a, hipStream_t stream);   // any supported shape
hipError_t launch_combine(const AttnArgs& a, hipStream_t stream);
bool general_supports(int Dqk, int Dv);
bool gqa128_supports(const AttnArgs& a);                            // D = 128, pages of 16..1024 tokens (power of two)
hipError_t launch_gqa128(const AttnArgs& a, hipStream_t stream);
bool mla_supports(const AttnArgs& a);                               // shared latent 576/512, pages of 32..1024 tokens
hipError_t launch_mla(const AttnArgs& a, hipStream_t stream);
hipError_t launch_short(const AttnArgs& a, hipStream_t stream);     // calls of short_call
hipError_t launch_tile(const AttnArgs& a, hipStream_t stream);      // shapes of tile_supports

}  // namespace seer
