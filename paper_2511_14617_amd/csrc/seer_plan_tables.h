// The plan's tables, as a workgroup writes them for the kernels that follow it and for calls that reuse the plan.
#pragma once
#include "seer_attention.h"
#include "seer_device.h"
#include "seer_plan.h"

namespace seer {

constexpr int kPlanLdsRequests = 4096;   // tile offsets of this many requests are searched in LDS, of more in global memory

// The plan's second workgroup.  Leading pages that a request has in common with the request before or after it
// (the prompt that the rollouts of a group share sits in the same physical pages): the partition kernel loads such
// tiles with the cache policy that keeps them, so that the repeats are served by the memory-side cache.  This is a
// hint only, results do not depend on it, so the length of the common run is found by probing instead of comparing
// every entry: sixteen entries at doubling distances, then sixteen evenly spaced ones between the last equal probe
// and the first unequal one (two dependent rounds of loads; exact for runs of up to 32 pages, else short by less
// than a sixteenth of the run if the tables are equal up to a point and differ behind it).  It runs beside the
// first workgroup, which needs about as long for the tile line and the stretches.  (Spread over workgroups of eight requests
// the plan kernel takes longer, calls of 75 to 110 requests 1.8 .. 2.7 us: workgroups of sixteen waves are slow to start.)
__device__ __forceinline__ void plan_shared_pages(const AttnArgs& p, int b_begin, int b_end, int threads) {
    for (int b = b_begin + static_cast<int>(threadIdx.x); b < b_end; b += threads) {
        const int n = p.ctx_len[b];
        int best = 0;
        if (n >= p.T && n <= p.max_ctx) {
            const int32_t* mine = p.block_table + static_cast<size_t>(b) * p.max_pages;
            const int pages = (n + p.P - 1) / p.P;
            int m[2] = {0, 0};                 // entries that can be compared with the neighbour
            const int32_t* other[2] = {mine, mine};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int nb = s ? b + 1 : b - 1;
                if (nb < 0 || nb >= p.B) continue;
                const int nn = p.ctx_len[nb];
                if (nn < p.T || nn > p.max_ctx) continue;
                m[s] = min(pages, (nn + p.P - 1) / p.P);
                other[s] = p.block_table + static_cast<size_t>(nb) * p.max_pages;
            }
            uint32_t eq[2] = {0u, 0u};        // bit k: probe k found equal entries
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int i = (1 << k) - 1;
                    const int ic = min(i, max(m[s] - 1, 0));
                    eq[s] |= static_cast<uint32_t>((i < m[s]) & (mine[ic] == other[s][ic])) << k;
                }
            int lo[2], step[2], hi[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int k = __builtin_ctz(~eq[s]);          // first probe that differs or lies outside (<= 16)
                lo[s] = k ? (1 << (k - 1)) : 0;               // number of leading entries taken as equal
                hi[s] = k ? min((1 << k) - 1, m[s]) : 0;      // entry hi differs or does not exist
                step[s] = max(1, (hi[s] - lo[s] + 15) / 16);
                eq[s] = 0u;
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int i = lo[s] + (j + 1) * step[s] - 1;
                    const int ic = min(i, max(m[s] - 1, 0));
                    eq[s] |= static_cast<uint32_t>((i < hi[s]) & (mine[ic] == other[s][ic])) << j;
                }
#pragma unroll
            for (int s = 0; s < 2; ++s) best = max(best, min(lo[s] + __builtin_ctz(~eq[s]) * step[s], hi[s]));
        }
        const_cast<int32_t*>(p.shared_tiles)[b] = static_cast<int>(static_cast<long long>(best) * p.P / kPlanTile);
    }
}

template <int THREADS>
struct PlanLds {
    int tiles[THREADS / kWave], longest[THREADS / kWave];       // per wave
    int start[kMaxWgsPerHead + 1];
    int first[kWholeRequests], part[THREADS / kWave];      // first stretch of each request, where none goes on into the next; per wave
    int off[kPlanLdsRequests + 1];
};

// One workgroup turns ctx_len[B] into the tile line, the stretch of every partition workgroup and the partial slots of every
// request.  (A history is read by workgroups of at least kMaxWgsPerHead threads only: one stretch per thread.)
template <int THREADS>
__device__ __forceinline__ void plan_tables(const AttnArgs& p, PlanLds<THREADS>& lds) {
    int (&s_tiles)[THREADS / kWave] = lds.tiles;
    int (&s_longest)[THREADS / kWave] = lds.longest;
    int* const s_start = lds.start;
    int* const s_off = lds.off;
    int32_t* const tile_off = const_cast<int32_t*>(p.tile_off);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int W = p.wgs_per_head;
    const bool balanced = p.balanced != 0, history = balanced && !p.fixed_split;
    const bool in_lds = p.B <= kPlanLdsRequests;

    // ---- everything this thread reads from global memory: its run of requests (one each up to 1024), its stretch -----
    const int per = (p.B + THREADS - 1) / THREADS;
    const int b0 = min(p.B, tid * per), b1 = min(p.B, b0 + per);
    const int n_first = b0 < b1 ? p.ctx_len[b0] : 0;
    uint32_t before = equal_before(p, tid), recorded = 0u;
    bool marked = true, usable = false;                  // is there a history; can it be used, as far as this thread's stretch goes
    if (history) {
        const uint32_t magic = p.header->fb_magic;
        const int w = p.header->fb_w;
        recorded = p.fb_before[min(tid, W)];
        const uint32_t behind = p.fb_before[min(tid, W) + 1];
        marked = magic == kFeedbackMagic && w == W;
        usable = marked && share_ok(p, tid, recorded, behind);
    }
    // a new one begins with this call's measurements
    if (!marked && tid < W) p.fb_time[tid] = 0u, p.fb_tiles[tid] = 0u, p.fb_speed[tid] = 0.f;
    auto tiles = [&](int n) -> int { return tiles_of(n, p.T, p.max_ctx); };
    auto length = [&](int b) -> int { return b == b0 ? n_first : p.ctx_len[b]; };

    // ---- sums inside the wave: tiles of its requests --------------------------------------------------------------------
    int cnt = 0, mx = 0;
    bool bad = false;
    for (int b = b0; b < b1; ++b) {
        const int n = length(b), t = tiles(n);
        bad |= n < p.T || n > p.max_ctx;                 // flagged, gets a zero output
        cnt += t;
        mx = max(mx, t);
    }
    const int incl = wave_incl_scan(cnt);
    const int wave_bad = __any(bad) ? 1 : 0;
    const bool wave_usable = __all(usable);
    mx = wave_max_in_last_lane(mx);
    if (lane == kWave - 1) {
        s_tiles[wave] = incl;
        s_longest[wave] = mx * 4 + (wave_usable ? 2 : 0) + wave_bad;
    }
    __syncthreads();
    int total = 0, my_off = incl - cnt, longest = 0;
    int any_bad = 0, all_usable = 2;
#pragma unroll
    for (int w = 0; w < THREADS / kWave; ++w) {
        const int t = s_tiles[w], l = s_longest[w];
        if (w < wave) my_off += t;
        total += t;
        longest = max(longest, l >> 2);
        any_bad |= l & 1;
        all_usable &= l & 2;
    }
    if (all_usable) before = recorded;
    {
        int off = my_off;
        for (int b = b0; b < b1; ++b) {
            tile_off[b] = off;
            if (in_lds) s_off[b] = off;
            off += tiles(length(b));
        }
        if (tid == 0) {
            tile_off[p.B] = total;
            if (in_lds) s_off[p.B] = total;
        }
    }

    if (balanced) {
        // ---- the stretches ----------------------------------------------------------------------------------------------
        Cut cut = cut_of(p, total, longest);
        static_assert(kSelfPlanRequests <= kWholeRequests && kWholeRequests <= THREADS, "both planners cut alike; one request per thread");
        const bool short_line = !cut.weighted && cut.equal > 1 && p.B <= kWholeRequests;
        int used = W + 1;
        if (short_line) {
            Cut tried = cut;
            for (const int most = longest_whole(cut); tried.equal <= most && used > W; ++tried.equal) {
                const int own = stretches_of(tried, cnt), incl_own = wave_incl_scan(own);
                if (lane == kWave - 1) lds.part[wave] = incl_own;
                __syncthreads();
                int in_front = incl_own - own;
                used = 0;
#pragma unroll
                for (int w = 0; w < THREADS / kWave; ++w) {
                    if (w < wave) in_front += lds.part[w];
                    used += lds.part[w];
                }
                if (used <= W) cut.equal = tried.equal;
                if (tid < p.B) lds.first[tid] = in_front;
                __syncthreads();
            }
        }
        if (used <= W) {
            for (int w = tid; w < W; w += THREADS) {
                int lo = 0, hi = p.B - 1;                // the last request whose stretches start at or before w
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (lds.first[mid] <= w) lo = mid; else hi = mid - 1;
                }
                const int size = s_off[lo + 1] - s_off[lo];
                s_start[w] = s_off[lo] + min(min(w - lds.first[lo], stretches_of(cut, size)) * cut.equal, size);
            }
        } else {
            for (int w = tid; w < W; w += THREADS) s_start[w] = cut_begin(cut, w, w == tid ? before : equal_before(p, w));
        }
        if (tid == 0) s_start[W] = total;
    }
    __syncthreads();

    // ---- per stretch: where it starts ------------------------------------------------------------------------------------
    for (int w = tid; w < W; w += THREADS) {
        StretchRec r;
        auto off = [&](int b) -> int { return in_lds ? s_off[b] : tile_off[b]; };
        if (balanced) {
            r.tile_begin = s_start[w], r.tile_end = s_start[w + 1];
            r.b = -1, r.req_begin = 0;
            if (r.tile_begin < r.tile_end) {             // the last request that starts at or before the first tile
                int lo = 0, hi = p.B - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (off(mid) <= r.tile_begin) lo = mid; else hi = mid - 1;
                }
                r.b = lo;
                r.req_begin = off(lo);
            }
        } else {
            r.tile_begin = off(w), r.tile_end = off(w + 1);
            r.req_begin = r.tile_begin;
            r.b = r.tile_begin < r.tile_end ? w : -1;
        }
        const_cast<StretchRec*>(p.stretch)[w] = r;
    }
    // ---- per request: its partial slots ----------------------------------------------------------------------------------
    // stretch that holds tile x (x < total): the last one that starts at or before it
    auto stretch_of = [&](int x) -> int {
        int lo = 0, hi = W - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_start[mid] <= x) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    int lo = my_off;
    for (int b = b0; b < b1; ++b) {
        const int hi = lo + tiles(length(b));
        ReqSlots s{0, -1};
        if (hi > lo) {
            const int first = balanced ? stretch_of(lo) : 0;
            s.first = first + b;
            s.last = (balanced ? stretch_of(hi - 1) : 0) + b;
        }
        const_cast<ReqSlots*>(p.req_slots)[b] = s;
        lo = hi;
    }
    if (tid == 0) {
        p.header->status = any_bad ? 1u : 0u;
        p.header->plan_b = plan_b_word(p.B);
        p.header->plan_w = plan_w_word(W, balanced);
        if (!marked) p.header->fb_magic = kFeedbackMagic, p.header->fb_w = W;
    }
}

}  // namespace seer
