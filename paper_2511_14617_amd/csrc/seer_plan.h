// The split of a call into stretches, as the plan kernel and the partition kernels that plan for themselves compute it.
#pragma once
#include "seer_attention.h"
#include "seer_device.h"

namespace seer {

// Inclusive sum over the lanes of a wave through DPP: shifts by 1, 2, 4, 8 inside rows of 16 lanes, then the last lane of a
// row to the row behind it and of the lower half to the upper (lanes without a source add zero).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_take(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, true); }
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += dpp_take<0x111, 0xf>(v);
    v += dpp_take<0x112, 0xf>(v);
    v += dpp_take<0x114, 0xf>(v);
    v += dpp_take<0x118, 0xf>(v);
    v += dpp_take<0x142, 0xa>(v);
    v += dpp_take<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ float wave_incl_scan(float v) {
    auto step = [&](int x) { v += __int_as_float(x); };
    step(dpp_take<0x111, 0xf>(__float_as_int(v)));
    step(dpp_take<0x112, 0xf>(__float_as_int(v)));
    step(dpp_take<0x114, 0xf>(__float_as_int(v)));
    step(dpp_take<0x118, 0xf>(__float_as_int(v)));
    step(dpp_take<0x142, 0xa>(__float_as_int(v)));
    step(dpp_take<0x143, 0xc>(__float_as_int(v)));
    return v;
}
// Maximum of non-negative values over the wave, in its last lane (lanes without a source count as zero).
__device__ __forceinline__ int wave_max_in_last_lane(int v) {
    v = max(v, dpp_take<0x111, 0xf>(v));
    v = max(v, dpp_take<0x112, 0xf>(v));
    v = max(v, dpp_take<0x114, 0xf>(v));
    v = max(v, dpp_take<0x118, 0xf>(v));
    v = max(v, dpp_take<0x142, 0xa>(v));
    v = max(v, dpp_take<0x143, 0xc>(v));
    return v;
}
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, kWave - 1); }
__device__ __forceinline__ float last_lane(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1)); }

// Tiles of a request of n tokens (a length outside [T, max_ctx] is flagged and gets a zero output).
__device__ __forceinline__ int tiles_of(int n, int T, int max_ctx) { return n < T || n > max_ctx ? 0 : (n + kPlanTile - 1) / kPlanTile; }

// x / d for 0 <= x < 2^31 and 1 <= d, with inv = reciprocal(d).  (A division by a number in a register is some thirty
// instructions, and every workgroup begins with two; the code itself has to be fetched, too.)
__host__ __device__ __forceinline__ int divide(int x, int d, uint32_t inv) {
    int q = static_cast<int>((static_cast<uint64_t>(static_cast<uint32_t>(x)) * inv) >> 32);       // the quotient or one less
    return x - q * d >= d ? q + 1 : q;
}

// How a line of `total` tiles, whose longest request has `longest`, is cut into W stretches.
struct Cut {
    int total, W, equal;      // tiles of the line, stretches, tiles of a stretch where all are alike
    bool weighted;            // the line is long enough for stretches that follow the measured speeds
};
__host__ __device__ __forceinline__ Cut cut_of(const AttnArgs& a, int total, int longest) {
    const int W = a.wgs_per_head;
    // a request of t tiles touches at most ceil(t / Lmin) + 1 stretches, which must fit max_splits
    const int per_w = divide(total + W - 1, W, a.inv_wgs);
    const bool fine = per_w < 2 || per_w >= kMinTilesLatent || total <= static_cast<long long>(a.fine_pieces - a.B) * per_w;
    const int Lmin = max(fine ? a.min_tiles : kMinTilesLatent, divide(longest + a.max_splits - 2, a.max_splits - 1, a.inv_splits));
    // Stretch w begins at the tile nearest to total * (r_0 + .. + r_{w-1}) / R.  When the line is too
    // short for that to keep every stretch at Lmin tiles or more, cut it into equal stretches of
    // max(Lmin, ceil(total / W)) tiles instead (the last ones are then short or empty).
    return {total, W, max(Lmin, max(per_w, 1)), total >= static_cast<long long>(max(2 * Lmin, kMinTilesWeighted)) * W};
}
// First tile of stretch w; before = (r_0 + .. + r_{w-1}) / R in units of 2^-32 (looked at only where the cut is weighted).
__host__ __device__ __forceinline__ int cut_begin(const Cut& c, int w, uint32_t before) {
    if (w >= c.W) return c.total;
    const uint64_t at = c.weighted ? (static_cast<uint64_t>(static_cast<uint32_t>(c.total)) * before + (1u << 31)) >> 32
                                   : static_cast<uint64_t>(w) * static_cast<uint32_t>(c.equal);
    return static_cast<int>(at < static_cast<uint64_t>(c.total) ? at : c.total);
}
// A short line (equal stretches) of up to kWholeRequests requests is cut so that no stretch goes on into the next request, where
// that takes no more than W stretches: stretch first + i of a request begins i * c.equal tiles into it.  A second piece costs its workgroup
// more than a tile (query rows, a first tile to wait for, partial results of its own), and the call waits for the slowest: of 459 workgroups of
// three tiles of 256-wide heads those with one piece were done after 18 .. 20 us, those with two after 28 (16 requests of 2730 tokens,
// one KV head: 36.0 -> 32.3 us a call; 64-wide heads 27.9 -> 25.8; 75 of 150 tokens, D = 128, two KV heads, 30.7 -> 27.2).
constexpr int kWholeRequests = 256;
// (Where stretches of c.equal tiles are too many, stretches of one more are tried, if that is no more than a third: 80 requests of 64 .. 1500
// tokens on 256-wide heads, four tiles cut across requests 46.0 us, five not 43.5; 60 of 64 .. 2000 41.2, 35.7.)
__host__ __device__ __forceinline__ int stretches_of(const Cut& c, int tiles) { return (tiles + c.equal - 1) / c.equal; }
__host__ __device__ __forceinline__ int longest_whole(const Cut& c) { return c.equal + (c.equal >= 3 ? 1 : 0); }
// The same where no speeds are known: w / W.
__host__ __device__ __forceinline__ uint32_t equal_before(const AttnArgs& a, int w) { return static_cast<uint32_t>(w) * a.inv_wgs; }

// Can words w and w + 1 of the recorded shares belong to a cut?  The first share has nothing in front of it, the last ends with
// the line, and rates between 3/4 and 4/3 make a share of 9/16 to 16/9 of an equal one; taken from 1/2 to 15/8 here.  W differences of at most
// 15/8 of 2^32 / W each, modulo 2^32, can only add up to 2^32 - 1 without a wrap: where all W pass, the shares rise from 0, the stretches
// cover the line once, and every one has a part of it that is a share's, whatever bytes the workspace held.  (Looked at in full by every
// wave that cuts: a mark beside the sums says who wrote them, not what has become of them since.)  (W >= 2)
__host__ __device__ __forceinline__ bool share_ok(const AttnArgs& a, int w, uint32_t here, uint32_t behind) {
    if (w >= a.wgs_per_head) return true;
    if (w + 1 == a.wgs_per_head) behind = 0xffffffffu;
    const uint32_t equal = a.inv_wgs;
    return (w > 0 || here == 0) && behind - here - equal / 2 <= equal + equal / 4 + equal / 8;
}

// ---------------------------------------------------------------------------
// A partition kernel's own plan.  A batch of up to kSelfPlanRequests requests has its lengths in one register of a wave, so
// every wave finds its stretch by itself: lengths and speeds in one round of loads, a scan over the lanes, one ballot.
// That takes the place of the load of the stretch's record; the plan kernel and its launch, 5.3 .. 5.8 us in front of
// every call, are not needed.  The tables that the combine kernel and calls which reuse the plan read are written by the workgroups
// of the first KV head and row block, each its own part.  (Larger batches would need several requests per lane and keep the kernel.)
// ---------------------------------------------------------------------------
constexpr int kLineWords = 2 * kSelfPlanRequests + 2;      // LDS: (first tile, tokens) per request, then (all tiles, -)

struct SelfPlan {
    StretchRec rec;
    int pieces;               // requests from the stretch's first to its last, those without tiles included (as the tables give it)
    bool new_history;         // the workspace holds none: this call begins it (see record_speed)
};
__device__ __forceinline__ SelfPlan plan_stretch(const AttnArgs& a, int* line, int wg) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1), W = a.wgs_per_head;
    const int n = lane < a.B ? a.ctx_len[lane] : 0;
    // the history: this stretch's two words, and eight words per lane to see whether all of them can be used
    struct Shares {
        u32x4 x, y;
        uint32_t next;
    };
    auto shares = [&](int i) __attribute__((always_inline)) -> Shares {          // i <= kMaxWgsPerHead - 8
        return {*reinterpret_cast<const u32x4*>(a.fb_before + i), *reinterpret_cast<const u32x4*>(a.fb_before + i + 4), a.fb_before[i + 8]};
    };
    static_assert(kMaxWgsPerHead % (8 * kWave) == 0 && kHistoryStride > kMaxWgsPerHead, "shares() stays inside the array");
    Shares s{};
    uint32_t f0 = 0u, f1 = 0u;
    bool usable = false, marked = true;
    if (!a.fixed_split) {
        usable = marked = a.header->fb_magic == kFeedbackMagic && a.header->fb_w == W;
        f0 = a.fb_before[wg], f1 = a.fb_before[wg + 1];
        s = shares(8 * lane);
    }
    const int t = lane < a.B ? tiles_of(n, a.T, a.max_ctx) : 0;
    const int incl = wave_incl_scan(t), off = incl - t;
    const int total = last_lane(incl), longest = last_lane(wave_max_in_last_lane(t));
    Cut cut = cut_of(a, total, longest);
    uint32_t before = equal_before(a, wg), behind = equal_before(a, wg + 1);
    if (!a.fixed_split && cut.weighted) {
        for (int i = 8 * lane;; s = shares(i)) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                usable &= share_ok(a, i + k, k < 4 ? s.x[k & 3] : s.y[k & 3], k < 3 ? s.x[(k + 1) & 3] : (k < 7 ? s.y[(k + 1) & 3] : s.next));
            i += 8 * kWave;
            if (i >= W) break;
        }
        if (__all(usable)) before = f0, behind = f1;
    }
    int begin, end;
    int own = 0, own_incl = 0;
    bool whole = false;
    if (!cut.weighted && cut.equal > 1) {       // (single tiles end with their request anyway)
        Cut tried = cut;
        for (const int most = longest_whole(cut); tried.equal <= most && !whole; ++tried.equal) {
            own = stretches_of(tried, t), own_incl = wave_incl_scan(own);
            whole = last_lane(own_incl) <= W;
            if (whole) cut.equal = tried.equal;
        }
    }
    if (whole) {
        const int first = own_incl - own, b = __popcll(__ballot(lane < a.B && first <= wg)) - 1;      // (the last one that starts at or before it)
        const int at = min(wg - __builtin_amdgcn_readlane(first, b), __builtin_amdgcn_readlane(own, b)) * cut.equal, size = __builtin_amdgcn_readlane(t, b);
        begin = __builtin_amdgcn_readlane(off, b) + min(at, size);
        end = __builtin_amdgcn_readlane(off, b) + min(at + cut.equal, size);
    } else {
        begin = __builtin_amdgcn_readfirstlane(cut_begin(cut, wg, before));
        end = __builtin_amdgcn_readfirstlane(cut_begin(cut, wg + 1, behind));
    }
    // every wave writes the same words and reads them behind its own writes
    line[2 * lane] = off, line[2 * lane + 1] = n;
    if (lane == 0) line[2 * kSelfPlanRequests] = total;
    SelfPlan r{{-1, begin, end, 0}, 1, !marked};
    if (begin < end) {                          // the last request that starts at or before the first tile
        r.rec.b = max(__popcll(__ballot(lane < a.B && off <= begin)) - 1, 0);
        r.rec.req_begin = __builtin_amdgcn_readlane(off, r.rec.b);
        int last = a.B - 1;
        if (end < total) {                      // the request that the next stretch starts in, if it does not start with it
            last = __popcll(__ballot(lane < a.B && off <= end)) - 1;
            if (__builtin_amdgcn_readlane(off, last) == end) --last;
        }
        r.pieces = max(1, last - r.rec.b + 1);
    }
    return r;
}

// At a wave's end (stores in front of its loads would have to be waited for with them): whether it met a page id outside the
// pool, one byte per wave of the grid (the status word cannot collect these: nothing in front of the kernel clears it); and by
// one workgroup per stretch that stretch's part of the tables.  (The stretches cover the line once, whatever the history held, so
// every request with tiles gets both words of its slots.)
__device__ __forceinline__ void publish_stretch(const AttnArgs& a, const int* line, const StretchRec& rec, int wg, int kvh, int rb, int wave,
                                                bool bad_page) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
    const bool any_bad = __any(bad_page);
    if (lane == 0) a.page_flags[((static_cast<size_t>(wg) * a.Hkv + kvh) * a.row_blocks + rb) * 8 + wave] = any_bad ? 1 : 0;
    if (kvh != 0 || rb != 0 || wave != 0) return;
    if (lane == 0) *const_cast<int4*>(reinterpret_cast<const int4*>(a.stretch + wg)) = make_int4(rec.b, rec.tile_begin, rec.tile_end, rec.req_begin);
    if (lane < a.B) {
        const int off = line[2 * lane], t = tiles_of(line[2 * lane + 1], a.T, a.max_ctx), last = off + t - 1;
        ReqSlots* slots = const_cast<ReqSlots*>(a.req_slots) + lane;
        if (t > 0 && off >= rec.tile_begin && off < rec.tile_end) slots->first = wg + lane;
        if (t > 0 && last >= rec.tile_begin && last < rec.tile_end) slots->last = wg + lane;
        if (wg == 0) {
            if (t == 0) *slots = ReqSlots{0, -1};
            const_cast<int32_t*>(a.tile_off)[lane] = off;
        }
    }
    if (wg == 0 && lane == 0) {
        const_cast<int32_t*>(a.tile_off)[a.B] = line[2 * kSelfPlanRequests];
        a.header->plan_b = plan_b_word(a.B);
        a.header->plan_w = plan_w_word(a.wgs_per_head, true);
    }
}

// At the end of a workgroup that had tiles, or of one without in a call that plans for itself, by one thread: its part of the speed history.
// set: the counters hold anything (a call that plans for itself, with nothing in front of it that could clear them, has found no
// history): the workgroup of the first KV head and row block sets them.
__device__ __forceinline__ void record_speed(const AttnArgs& a, int wg, int kvh, int rb, uint64_t ticks, int tiles, bool set) {
    const uint32_t t = static_cast<uint32_t>(ticks > 0xffffffu ? 0xffffffu : ticks);
    if (!set) {
        atomicAdd(a.fb_time + wg, t);
        atomicAdd(a.fb_tiles + wg, static_cast<uint32_t>(tiles));
    } else if (kvh == 0 && rb == 0) {
        a.fb_time[wg] = t;
        a.fb_tiles[wg] = static_cast<uint32_t>(tiles);
    }
}

// What a piece needs of request b: lanes 0, 1, 2 get its first tile, the first tile behind it, its tokens.  (Read and wait in one
// block: the compiler would put a wait for all tile loads in front of a read of its own.)
__device__ __forceinline__ int line_words(const int* line, int b) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
    const int word = 2 * b + (lane == 1 ? 2 : (lane == 2 ? 1 : 0));
    const int at = static_cast<int>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) int*)(line))) + 4 * word;
    int v;
    asm volatile("ds_read_b32 %0, %1\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v)
                 : "v"(at)
                 : "memory");
    return v;
}

// Pages, from page `first` of request b on, that a neighbouring request maps too: what shared_tiles says, found from the rows
// themselves, in the 64 pages that a piece begins with.  A hint like that table (entries behind a neighbour's end may be anything).
struct NeighbourRows {
    int above, below;         // each lane's entry of the requests in front and behind
};
__device__ __forceinline__ NeighbourRows neighbour_entries(const AttnArgs& a, int b, int page) {
    const int32_t* col = a.block_table + min(page, a.max_pages - 1);
    return {col[static_cast<size_t>(max(min(b, a.B) - 1, 0)) * a.max_pages], col[static_cast<size_t>(min(b + 1, a.B - 1)) * a.max_pages]};
}
// lane l: entry first + l
__device__ __forceinline__ NeighbourRows neighbour_rows(const AttnArgs& a, int b, int first) {
    return neighbour_entries(a, b, first + (static_cast<int>(threadIdx.x) & (kWave - 1)));
}
// Entries, in the order of the lanes, that request b and a neighbour have in common; mine: the lane's entry of request b.
__device__ __forceinline__ int shared_run(const AttnArgs& a, int b, int mine, const NeighbourRows& rows) {
    const uint64_t up = b > 0 ? ~__ballot(mine == rows.above) : ~0ull, down = b + 1 < a.B ? ~__ballot(mine == rows.below) : ~0ull;
    return up == 0 || down == 0 ? kWave : max(__builtin_ctzll(up), __builtin_ctzll(down));
}
// The run behind a window that is shared throughout, as far as the piece goes (its last page: `last`): one round of 64 evenly spaced
// probes, so exact for 64 further pages and short by less than a 64th of the rest beyond that.  (Window after window, and to the end of
// the row instead of the piece's, 64 requests on one KV head with common prompts of 32768 tokens took 189 us, 8 requests on two
// 60.5; now 177 and 51.2.)
__device__ __forceinline__ int shared_run_behind(const AttnArgs& a, int b, int first, int last) {
    const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
    const int count = last - first + 1;
    if (count <= 0) return 0;
    const int step = (count + kWave - 1) / kWave;
    const int page = first + min((lane + 1) * step, count) - 1;
    const int mine = a.block_table[static_cast<size_t>(b) * a.max_pages + min(page, a.max_pages - 1)];
    return min(shared_run(a, b, mine, neighbour_entries(a, b, page)) * step, count);
}

}  // namespace seer
