// seer_draft: grouped n-gram drafting, the step right before verification.
//
// What is computed (Section 2.3, pattern level; Section 3.4.2; Appendix A.2, draft client, call
// batch_speculate with SpeculationArgs max_spec_tokens / pattern_lookup_max / pattern_lookup_min /
// top_k): a request's draft tokens come from the token histories of all requests of its prompt
// group.  The request's newest tokens are the pattern; the longest pattern suffix that occurs in a
// history followed by at least one more token is the match; every continuation string of the
// match is a candidate path whose confidence is (places where match + path occurs) / (places
// where the match occurs with a continuation), i.e. the product of the conditional frequencies
// along the path; candidates below min_confidence are dropped and a beam search of width top_k
// returns several paths.  The paper keeps the histories in a compressed suffix tree that a
// separate server updates; here nothing is indexed: the histories are plain token arrays in HBM
// (appending a token is one store), and a lookup scans the group's history, which at 8 TB/s and
// with the group's tokens resident in L2 after the first request costs less than the tree's
// upkeep would.  Two kernels:
//
//   draft_match_kernel   grid (stretches, groups): a workgroup reads one stretch of a group's tokens
//                        once and, for every request of the group, measures at every place how many
//                        of the request's newest tokens end there; the places that reach the
//                        stretch's running maximum go to the request's place list
//   draft_expand_kernel  grid (requests): takes the longest match over all stretches, gathers its
//                        places, then searches level by level: the (member, next token) pairs of
//                        the live places are counted, the top_k picked, the places reassigned.
//                        The places' next tokens are held as strings, equal ones as one where places
//                        are many; more than that takes two lists in global memory.
//
// Counts are integers, the order of the beam is (count descending, parent rank ascending, token
// ascending) and the confidence test is one fp32 product and one comparison, so the result is
// unique and does not depend on the order in which places are found or atomics land.
//
// Both kernels are bound by the length of their dependent chains (a global round trip, an LDS round
// trip, a barrier), not by bandwidth: loads are requested in batches from addresses clamped into
// the pool and selected afterwards, so that a thread waits once per batch, not once per load.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/seer_verify.h"

namespace seer {
namespace draft {

constexpr int kMatchThreads = 256;        // match workgroup
constexpr int kThreads = 1024;            // expansion workgroup
constexpr int kMaxGroupSeqs = 128;        // sequences per group (7 bits of a place)
constexpr int kMaxSeqLenLog2 = 20;        // tokens per sequence < 2^20 (20 bits of a place)
constexpr int kMaxPattern = 32;           // pattern_lookup_max (5 bits of a place hold match length - 1)
constexpr int kMaxTopK = 16;
constexpr int kTableSlots = 4096;         // LDS hash table: 4096 x (key, count) = 32 KB
constexpr uint32_t kEmpty = 0xffffffffu;
constexpr int kMaxParts = 256;            // stretches a group's tokens are cut into, at most
constexpr int kReqWindow = 64;            // request ids a match workgroup looks at per round
// 16-byte loads a match thread has in flight.  Two (2048 tokens a workgroup): the per-request part of the scan is a chain whose
// length grows with the tokens a thread holds, and the launch has workgroups to spare (whole call, 16 requests of 6 k tokens
// 44.5 us with four, 37.7 with two, 36.4 with one; 128 requests, four paths: 126, 121, 125).
constexpr int kQuads = 2;
constexpr int kSet = 64 / (4 * kQuads);   // requests whose candidate places a thread notes at a time, a bit each
constexpr int kTile = 4 * kQuads * kMatchThreads;   // tokens a match workgroup takes per round
constexpr int kTokensPerPart = kTile;     // target length of a stretch: one round
constexpr int kSmall = 2048;              // up to this many places the expansion holds in registers
constexpr int kAhead = 8;                 // levels whose tokens it fetches at a time

// A place = (sequence inside the group, offset of the token that follows the occurrence); while the
// match is still being searched it also carries the match length.
__device__ __forceinline__ uint32_t pack_place(int seq, int m, int off) {
    return (static_cast<uint32_t>(seq) << 25) | (static_cast<uint32_t>(m - 1) << 20) | static_cast<uint32_t>(off);
}
__device__ __forceinline__ int place_seq(uint32_t e) { return static_cast<int>(e >> 25); }
__device__ __forceinline__ int place_len(uint32_t e) { return static_cast<int>((e >> 20) & 31u) + 1; }
__device__ __forceinline__ int place_off(uint32_t e) { return static_cast<int>(e & ((1u << kMaxSeqLenLog2) - 1)); }

struct Args {
    const int32_t* tokens;
    const int32_t* seq_start;
    const int32_t* seq_len;
    const int32_t* group_first;
    const int32_t* req_group;
    const int32_t* pattern;
    const int32_t* pattern_len;
    const int32_t* max_spec_tokens;
    int32_t* draft_tokens;
    int32_t* tree_parent;
    uint64_t* tree_mask;
    int32_t* node_count;        // may be nullptr
    int32_t* match_len;         // may be nullptr
    int32_t* status;            // may be nullptr
    int2* part_hdr;             // [B, parts] (places kept, longest match) of each match workgroup
    uint32_t* list_a;           // [B, cap]
    uint32_t* list_b;           // [B, cap]
    int64_t pool_tokens;
    int n_groups, n_seq, max_group_tokens;
    int gamma_max, top_k, p_min, p_max, vocab;
    int parts, chunk, cap;      // cap = parts * chunk >= max_group_tokens
    float min_confidence;
};

// What is the same in all lanes, where the compiler cannot know (words in LDS): in a scalar register, so that loops and
// branches on it are scalar ones.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int lane_id() { return static_cast<int>(threadIdx.x) & 63; }

// Index for each lane whose `hit` is set, from a counter in LDS: one atomic per wave instead of one per lane.
__device__ __forceinline__ int wave_append(int* counter, bool hit) {
    const uint64_t mask = __ballot(hit);
    if (mask == 0) return 0;
    const int leader = __ffsll(static_cast<long long>(mask)) - 1;
    int base = 0;
    if (lane_id() == leader) base = atomicAdd(counter, __popcll(mask));
    base = __builtin_amdgcn_readlane(base, leader);
    return base + __popcll(mask & ((1ull << lane_id()) - 1));
}

// The group's sequence table in LDS; n_seq = 0 and bad != 0 if it cannot be used.
struct GroupTable {
    int start[kMaxGroupSeqs];
    int len[kMaxGroupSeqs];
    int flat[kMaxGroupSeqs + 1];          // tokens of the group before sequence j
    int n_seq;
    int bad;
};

// By one wave (every lane of it calls; the caller has the barrier behind it), two sequences per lane: other waves use
// the three dependent loads' time for what does not depend on them.
static_assert(kMaxGroupSeqs == 128, "two sequences per lane");
__device__ __forceinline__ void load_group(const Args& a, int g, GroupTable& gt) {
    const int lane = lane_id();
    int bad = 0, q0 = 0, q1 = 0;
    if (g < 0 || g >= a.n_groups) {
        bad = 1;
    } else {
        q0 = a.group_first[g];
        q1 = a.group_first[g + 1];
        if (q0 < 0 || q1 < q0 || q1 > a.n_seq || q1 - q0 > kMaxGroupSeqs) {
            bad = 1;
            q1 = q0 = 0;
        }
    }
    const int n = q1 - q0;
    int st[2], ln[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int j = 2 * lane + k;
        st[k] = ln[k] = 0;
        if (j < n) st[k] = a.seq_start[q0 + j], ln[k] = a.seq_len[q0 + j];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (st[k] < 0 || ln[k] < 0 || ln[k] >= (1 << kMaxSeqLenLog2) || static_cast<int64_t>(st[k]) + ln[k] > a.pool_tokens)
            bad = 1, st[k] = ln[k] = 0;
    const int sum = ln[0] + ln[1];                // tokens of the group before a sequence (lengths are below 2^20)
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int before[2] = {incl - sum, incl - ln[1]};
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (2 * lane + k < n) gt.start[2 * lane + k] = st[k], gt.len[2 * lane + k] = ln[k], gt.flat[2 * lane + k] = before[k];
    bad = (__ballot(bad != 0) != 0 ? 1 : 0) | (total > a.max_group_tokens ? 2 : 0);
    if (lane == 0) gt.flat[n] = total, gt.bad = bad, gt.n_seq = bad ? 0 : n;
}

// ------------------------------------------------------------------------------------------------
// Match: how many pattern tokens end at each place of one stretch of a group's tokens, for every
// request of the group at once (the stretch is read once, whatever the number of requests).
// ------------------------------------------------------------------------------------------------
struct MatchShared {
    GroupTable gt;
    __attribute__((aligned(16))) int tile[kMaxPattern + kTile];   // the tokens before the tile, then the tile
    int pat[kReqWindow][kMaxPattern];
    int req[kReqWindow], plen[kReqWindow], best[kReqWindow], kept[kReqWindow];
    int4 info[kReqWindow + 1];                     // (newest token, the one before it, pattern length, -) per request
    int4 older[kReqWindow + 1];                    // the four pattern tokens before those two
    int n_req;
    int first_seq;                                 // the sequence that holds the first token a tile needs
};

// A tile is a run of kTile places of the group's tokens counted through all its sequences one after the
// other ("flat" positions), so a workgroup takes its whole stretch in one round however many sequences it
// touches.  No match runs from one sequence into the next: a place's match is bounded by its distance
// from the start of its own sequence.
__global__ __launch_bounds__(kMatchThreads) void draft_match_kernel(Args a, int B) {
    __shared__ MatchShared sh;
    const int g = blockIdx.y, part = blockIdx.x, tid = threadIdx.x;
    // The second wave takes the requests of this group among the kReqWindow consecutive ids from b0 on; for the first window
    // while the first wave waits for the group's table.
    auto take_requests = [&](int b0) __attribute__((always_inline)) {
        const int lane = lane_id(), b = b0 + lane;
        const int len = b < B ? a.pattern_len[b] : 0;
        const bool mine = b < B && a.req_group[b] == g;
        const uint64_t mask = __ballot(mine);
        if (mine) {
            const int r = __popcll(mask & ((1ull << lane) - 1));
            sh.req[r] = b;
            sh.plen[r] = min(max(len, 0), a.p_max);
            sh.best[r] = max(a.p_min, 1), sh.kept[r] = 0;
        }
        if (lane == 0) sh.n_req = __popcll(mask);
    };
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    if (wave == 0) load_group(a, g, sh.gt);
    if (wave == 1) take_requests(0);
    __syncthreads();
    const int need = max(a.p_min, 1);
    const bool two = need >= 2;
    const int n_seq = sh.gt.n_seq;
    const int total = n_seq > 0 ? sh.gt.flat[n_seq] : 0;
    const int lo = part * a.chunk, hi = min(lo + a.chunk, total);
    // requests are taken in windows of kReqWindow consecutive ids: at most that many belong to this group
    for (int b0 = 0; b0 < B; b0 += kReqWindow) {
        if (b0 > 0) {
            __syncthreads();                                        // (a window without requests has none behind its n_req)
            if (wave == 1) take_requests(b0);
            __syncthreads();
        }
        const int n_req = sh.n_req;
        if (n_req == 0) continue;
        for (int i = tid; i < n_req * a.p_max; i += kMatchThreads) {
            const int r = i / a.p_max, c = i - r * a.p_max;
            sh.pat[r][c] = a.pattern[static_cast<size_t>(sh.req[r]) * a.p_max + c];
        }
        __syncthreads();
        if (tid <= n_req) {
            auto back = [&](int k) { return tid < n_req && a.p_max > k ? sh.pat[tid][a.p_max - 1 - k] : 0; };
            sh.info[tid] = make_int4(back(0), back(1), tid < n_req ? sh.plen[tid] : 0, 0);
            sh.older[tid] = make_int4(back(2), back(3), back(4), back(5));
        }
        for (int t0 = lo; t0 < hi; t0 += kTile) {
            const int t1 = min(t0 + kTile, hi);                    // places of this tile: [t0, t1)
            const int halo0 = max(t0 - kMaxPattern, 0);            // first flat position the tile needs
            if (tid < n_seq && sh.gt.flat[tid] <= halo0 && halo0 < sh.gt.flat[tid + 1]) sh.first_seq = tid;
            __syncthreads();                                        // also: the previous tile is no longer read
            // Loads: for every sequence that reaches into the tile, each thread requests its 8 places (two
            // quads) and one token of the run before the tile, all from addresses clamped into the pool, then
            // keeps those that belong to the sequence.
            int tok[4 * kQuads];
#pragma unroll
            for (int c = 0; c < 4 * kQuads; ++c) tok[c] = 0;
            int before = 0;
            uint32_t inside = 0, has_prev = 0;                      // per place: may end a match; has a token before it
            for (int j = sh.first_seq; j < n_seq && sh.gt.flat[j] < t1; ++j) {
                const int f0 = sh.gt.flat[j], f1 = sh.gt.flat[j + 1];
                const int at0 = sh.gt.start[j] - f0;                // pool index of flat position 0 of this sequence
                int got[4 * kQuads];
#pragma unroll
                for (int c = 0; c < 4 * kQuads; ++c) {
                    const int p = t0 + 4 * tid + (c >> 2) * 4 * kMatchThreads + (c & 3);
                    const bool in = p >= f0 && p < f1 && p < t1;
                    got[c] = a.tokens[in ? at0 + p : 0];
                }
                const int ph = t0 - kMaxPattern + tid;
                const bool in_h = tid < kMaxPattern && ph >= f0 && ph < f1;
                const int got_h = a.tokens[in_h ? at0 + ph : 0];
#pragma unroll
                for (int c = 0; c < 4 * kQuads; ++c) {
                    const int p = t0 + 4 * tid + (c >> 2) * 4 * kMatchThreads + (c & 3);
                    const bool in = p >= f0 && p < f1 && p < t1;
                    tok[c] = in ? got[c] : tok[c];
                    if (in && p + 1 < f1) inside |= 1u << c;       // the token that follows exists
                    if (in && p > f0) has_prev |= 1u << c;
                }
                before = in_h ? got_h : before;
            }
            if (tid < kMaxPattern) sh.tile[tid] = before;
#pragma unroll
            for (int u = 0; u < kQuads; ++u)
                *reinterpret_cast<int4*>(&sh.tile[kMaxPattern + 4 * tid + u * 4 * kMatchThreads]) =
                    make_int4(tok[4 * u], tok[4 * u + 1], tok[4 * u + 2], tok[4 * u + 3]);
            __syncthreads();
            // the token before each of this thread's quads (the others are in its registers)
            int prev_quad[kQuads];
#pragma unroll
            for (int u = 0; u < kQuads; ++u) prev_quad[u] = sh.tile[kMaxPattern + 4 * tid + u * 4 * kMatchThreads - 1];
            // Requests go in sets of kSet: first, which of the thread's places end a match of at least `need` tokens for which
            // request, a bit each, from registers; then every lane that has such places takes one of them per round,
            // whatever its request (round after round per request, most of them with a lane or two, the scan took 13.1 us
            // for 16 requests in two groups and 18.2 for 128 in sixteen; now 11.6 and 16.0).
            int4 info = sh.info[0];
            for (int r0 = 0; r0 < n_req; r0 += kSet) {
                uint64_t hits = 0;
#pragma nounroll
                for (int k = 0; k < min(kSet, n_req - r0); ++k) {
                    // A place counts only if at least `need` pattern tokens end there: with need >= 2 the token
                    // before it is tested too, in registers, which leaves few places to look at closely.
                    // (The next request's constants are requested before this one's are used.)
                    const int newest = info.x, second = info.y, plen = info.z;
                    info = sh.info[r0 + k + 1];
                    if (plen < need) continue;
                    // first only whether any lane holds a candidate at all: two compares per place
                    bool any = false;
#pragma unroll
                    for (int c = 0; c < 4 * kQuads; ++c) {
                        const int prev = (c & 3) ? tok[c - 1] : prev_quad[c >> 2];
                        any |= (tok[c] == newest) & (!two | (prev == second));
                    }
                    if (__ballot(any) == 0) continue;
                    uint32_t set = 0;
#pragma unroll
                    for (int c = 0; c < 4 * kQuads; ++c) {
                        const int prev = (c & 3) ? tok[c - 1] : prev_quad[c >> 2];
                        bool h = tok[c] == newest && ((inside >> c) & 1u) != 0;
                        if (two) h = h && prev == second && ((has_prev >> c) & 1u) != 0;
                        set |= static_cast<uint32_t>(h) << c;
                    }
                    hits |= static_cast<uint64_t>(set) << (k * 4 * kQuads);
                }
                while (__ballot(hits != 0) != 0) {
                    if (hits == 0) continue;
                    const int bit = __builtin_ctzll(hits);
                    hits &= hits - 1;
                    const int r = r0 + bit / (4 * kQuads), c = bit & (4 * kQuads - 1);
                    const int p = t0 + 4 * tid + (c >> 2) * 4 * kMatchThreads + (c & 3);
                    const int4 mine = sh.info[r];
                    const int4 older = sh.older[r];
                    const int best = sh.best[r];
                    int j = sh.first_seq;                              // the sequence that holds place p
                    while (p >= sh.gt.flat[j + 1]) ++j;
                    const int off = p - sh.gt.flat[j];
                    const int limit = min(mine.z, off + 1);           // not past the start of the sequence
                    const int* at = &sh.tile[kMaxPattern + (p - t0)];
                    // the five tokens before the place are requested together and compared in registers;
                    // only a longer match goes on through LDS
                    const int v1 = at[-1], v2 = at[-2], v3 = at[-3], v4 = at[-4], v5 = at[-5];
                    int m = 1;
                    bool on = 1 < limit && v1 == mine.y;
                    m += on ? 1 : 0, on = on && 2 < limit && v2 == older.x;
                    m += on ? 1 : 0, on = on && 3 < limit && v3 == older.y;
                    m += on ? 1 : 0, on = on && 4 < limit && v4 == older.z;
                    m += on ? 1 : 0, on = on && 5 < limit && v5 == older.w;
                    m += on ? 1 : 0;
                    if (on)
                        while (m < limit && at[-m] == sh.pat[r][a.p_max - 1 - m]) ++m;
                    // a shorter match than one already seen in this stretch can never win
                    if (m < best) continue;
                    if (m > best) atomicMax(&sh.best[r], m);
                    const int slot = atomicAdd(&sh.kept[r], 1);
                    a.list_a[static_cast<size_t>(sh.req[r]) * a.cap + static_cast<size_t>(part) * a.chunk + slot] = pack_place(j, m, off + 1);
                }
            }
            __syncthreads();                                        // sh.first_seq and the tile are free again
        }
        __syncthreads();
        if (tid < n_req)
            a.part_hdr[static_cast<size_t>(sh.req[tid]) * a.parts + part] = make_int2(sh.kept[tid], sh.kept[tid] > 0 ? sh.best[tid] : 0);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// Expand: beam search over the continuations of the longest match.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    auto step = [&](auto ctrl) __attribute__((always_inline)) {
        const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), decltype(ctrl)::value, 0xf, 0xf, false));
        v = w > v ? w : v;
    };
    step(std::integral_constant<int, 0x111>{}), step(std::integral_constant<int, 0x112>{});     // row_shr 1, 2, 4, 8
    step(std::integral_constant<int, 0x114>{}), step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{}), step(std::integral_constant<int, 0x143>{});     // row_bcast 15, 31
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    const uint32_t hi = wave_max_u32(static_cast<uint32_t>(v >> 32));
    const uint32_t lo = wave_max_u32(static_cast<uint32_t>(v >> 32) == hi ? static_cast<uint32_t>(v) : 0u);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int lane) {
    return (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), lane))) << 32) |
           static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), lane));
}
__device__ __forceinline__ int wave_sum(int v) {
    auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
        v += __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{}), step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{}), step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}), step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
    return __builtin_amdgcn_readlane(v, 63);
}

struct Member {            // one beam member of the current level
    int base, n, slot;     // its places are list[base .. base + n) while the places live in global memory
};

// ---- up to kSmall places: the tokens that follow them, as strings in LDS, kAhead levels at a time ----
//
// What bounds the search is the chain of LDS round trips (some 130 clocks each) and of issued instructions of the request
// with the most places: an LDS atomic costs about a clock per lane, and an instruction of sixteen waves sixteen clocks.
// So as few strings as can be go through as little as can be:
//   - the levels on which all strings agree are settled at once;
//   - the lanes of a wave that show what its first one shows are settled inside the wave; where that says that most recur,
//     more than kFew places are reduced to distinct strings (a phrase that recurs a thousand times goes on in a
//     few dozen ways); a string that half of the places show stays once, however many there are;
//   - while more than a wave's worth of strings is left, a level counts its (member, token) pairs in a hash table
//     and the beam drops the strings nobody goes on with (most of them, where strings part); up to kFew strings are
//     four waves' work, up to twice as many eight waves', and the waves without work end;
//   - up to 64 strings, one per lane, are searched by one wave in registers: the lanes that show what the first one left
//     shows are one pair, found and counted with one ballot.
// When each level was counted by the whole workgroup behind six barriers (7 .. 12 thousand clocks a level with sixteen
// waves, 2 .. 3 thousand for one wave with up to 256 places), whole calls of 128 requests with four paths of eight over 16
// draws of the histories took 64 .. 212 us, 103 on average; 44 .. 74 and 52.5 now (16 of it the match scan); 300 requests
// 170 us, 95 now, 1024 of shorter histories 123, 92 now.  Slower than that are more than eight levels of one phrase (141 places: 27 us, 38
// now) and thousands of places with nearly as many strings over a few tokens (2450: 61, 74; 6701: 100, 125).
// The search takes 152,480 bytes of LDS, so one workgroup per CU; sixteen waves of up to 128 registers leave no room
// for a second one in any case.
// Not kept: comparing all strings with each other (n^2 / 64 wave steps of some 60 instructions) and a trie of all
// levels in one table (strings that the beam drops at the next level are entered all the way down).
constexpr int kSlots = 4096;              // of the table of a level's pairs, at most
constexpr int kFew = 512;
constexpr int kFewThreads = 256;
constexpr int kPer = kSmall / kThreads;   // strings per thread, at most
// Distinct strings stay distinct only as far as they are known: they are for the last kAhead levels, and cost what two
// or three levels of the table do (two levels, 1207 places with 691 strings: whole call 37.8 us with them, 36.0 without).
constexpr int kDistinctLevels = 3;
constexpr int kSettled = 4;               // so many strings settled inside their waves say that at least three in four recur
constexpr int kManyPlaces = 1 << 16;      // (numbers of places in 16 bits)
// More than kSmall places are given up after the first kThreads if as many in proportion would be this many distinct ones
// (later places repeat more; 2761 places with 2034 strings: whole call 155 us without the strings, 68 with; 3787 with 3058: 91, given up late 98).
constexpr int kHopeless = kSmall * 5 / 4;
constexpr int kRankWave = 16;             // candidates of a level that are ranked one by one
constexpr int kPeel = 4;                  // pairs that one wave takes one by one before it looks for the rest by hash
constexpr int kMeetLog2 = 9;              // words it uses for that
constexpr int kListed = 4;                // pairs of a longer list per lane and round
constexpr uint64_t kNoPair = ~0ull;       // an entry: strings << 48 | places << 32 | rank of the member << 24 | token
static_assert((4 << kMeetLog2) <= 2 * kSmall, "words in the list");
static_assert(kSlots >= 2 * kSmall && kFew <= kPer * kFewThreads, "strings per table and thread");

// What the expansion keeps in LDS.
struct Expand {
    GroupTable gt;
    union {
        struct {                           // while the places live in global memory: the pairs of a level
            uint32_t key[kTableSlots];
            uint32_t cnt[kTableSlots];
        };
        __attribute__((aligned(16))) int row[kSmall][kAhead];    // strings, while they change threads
        struct {                           // while distinct strings are found among more than kSmall places
            __attribute__((aligned(16))) int fresh[kThreads][kAhead];
            __attribute__((aligned(16))) int kept[kSmall][kAhead];
        };
        __attribute__((aligned(16))) uint64_t pair[2][kSlots];   // the pairs of a level, and the next level's cleared table
    };
    uint32_t distinct[2 * kSmall];         // while distinct strings are found
    int8_t rank[2][kSlots];                // of a pair among the level's picks, -1 = not picked
    uint16_t id[kSmall], weight[kSmall];   // of the strings that change threads: a place that shows it, how many do,
    int8_t member[kSmall];                 //   and the rank of the member it belongs to
    __attribute__((aligned(16))) uint16_t list[kSmall];          // entries of the level's pairs (in one wave's search, the words of its hash)
    int lead[kAhead], lead_member;         // the string that the others are compared with
    int n_list[2], n_held, n_left, common;
    uint32_t n_on;
    uint32_t place[kSmall];                // hand-over of places between the phases
    int8_t owner[kSmall];                  // rank of the member a place belongs to, -1 = dropped
    int first[kMaxParts + 1];              // places of the longest match before part p
    Member mem[kMaxTopK], next[kMaxTopK];  // members while the places live in global memory
    uint64_t red[kThreads / 64];
    int ref[kMaxTopK], ref_cnt[kMaxTopK];  // the token all places of a member show, and how many show it
    uint64_t pick[kMaxTopK];               // chosen children: count << 32 | ~key, best first
    int fill[kMaxTopK];
    int tok[SEER_MAX_T], par[SEER_MAX_T], num[SEER_MAX_T];
    uint64_t msk[SEER_MAX_T];
    int n, best_len, nmem, overflow;
};

// count[key] += n in the hash table (open addressing, linear probing).
__device__ __forceinline__ void hash_add(Expand& x, int table, int shift, uint32_t key, uint32_t n) {
    uint32_t h = (key * 2654435761u) >> shift;
    for (int probes = 0; probes < table; ++probes) {
        const uint32_t old = atomicCAS(&x.key[h], kEmpty, key);
        if (old == kEmpty || old == key) {
            atomicAdd(&x.cnt[h], n);
            return;
        }
        h = (h + 1) & (table - 1);
    }
    x.overflow = 1;
}

// Places in global memory: the first top_k table entries in the order (count descending, key ascending)
// that pass the confidence test join x.pick (kept sorted, best first, at most top_k long).  Every thread
// returns the new length.
__device__ __forceinline__ int pick_top(Expand& x, int slots, float threshold, int top_k, int n_pick) {
    const int tid = threadIdx.x;
    for (int round = 0; round < top_k; ++round) {
        uint64_t best = 0;
        for (int s = tid; s < slots; s += kThreads) {
            const uint32_t c = x.cnt[s];
            if (c == 0 || static_cast<float>(c) < threshold) continue;
            const uint64_t v = (static_cast<uint64_t>(c) << 32) | static_cast<uint32_t>(~x.key[s]);
            best = v > best ? v : best;
        }
        uint64_t win = wave_max_u64(best);
        if (lane_id() == 0) x.red[tid >> 6] = win;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) win = x.red[w] > win ? x.red[w] : win;
        if (win == 0) {
            __syncthreads();
            break;
        }
        const uint32_t win_key = ~static_cast<uint32_t>(win);
        for (int s = tid; s < slots; s += kThreads)
            if (x.key[s] == win_key) x.cnt[s] = 0;
        if (tid == 0) {
            int at = n_pick < top_k ? n_pick : top_k - 1;
            if (n_pick < top_k || win > x.pick[at]) {
                while (at > 0 && x.pick[at - 1] < win) {
                    x.pick[at] = x.pick[at - 1];
                    --at;
                }
                x.pick[at] = win;
            }
        }
        n_pick = min(n_pick + 1, top_k);
        __syncthreads();
    }
    return n_pick;
}

// Places in global memory: the picks of level d become draft nodes (one thread).
__device__ __forceinline__ void emit_nodes(Expand& x, int d, int top_k, int n_pick) {
    int base = 0;
    for (int j = 0; j < n_pick; ++j) {
        const uint32_t key = ~static_cast<uint32_t>(x.pick[j]);
        const int c = static_cast<int>(x.pick[j] >> 32), r = static_cast<int>(key >> 24);
        const int slot = 1 + (d - 1) * top_k + j, parent = x.mem[r].slot;
        x.tok[slot] = static_cast<int>(key & 0xffffffu);
        x.par[slot] = parent;
        x.num[slot] = c;
        x.msk[slot] = (1ull << slot) | x.msk[parent];
        x.next[j] = Member{base, c, slot};            // x.mem is still needed until the places are reassigned
        x.fill[j] = 0;
        base += c;
    }
}

// Slot of the member of this rank at the level before d (the root in front of the first level).
__device__ __forceinline__ int member_slot(int d, int top_k, int rank) { return d == 1 ? 0 : 1 + (d - 2) * top_k + rank; }

// Draft node of rank `rank` at level d, for the pick `val` (count << 32 | ~key).
__device__ __forceinline__ void put_node(Expand& x, int d, int top_k, int rank, uint64_t val) {
    const uint32_t key = ~static_cast<uint32_t>(val);
    const int slot = 1 + (d - 1) * top_k + rank, parent = member_slot(d, top_k, static_cast<int>(key >> 24));
    x.tok[slot] = static_cast<int>(key & 0xffffffu);
    x.par[slot] = parent;
    x.num[slot] = static_cast<int>(val >> 32);
    x.msk[slot] = (1ull << slot) | x.msk[parent];
}

// What a thread holds: strings (their words still to be searched in front, -1 behind their end), a place that shows
// each, how many do, and the rank of the member it belongs to (-1: nobody goes on with it).
struct Held {
    int t[kPer][kAhead], id[kPer], w[kPer], member[kPer];
};

// The words of a place's string from level d on, at most L: requested (returns how many there are), and as a string: -1 behind its
// end, or if the place belongs to nobody.
__device__ __forceinline__ int request_string(const Args& a, const Expand& x, uint32_t place, bool on, int d, int L, int (&t)[kAhead]) {
    const int j = place_seq(place), off = place_off(place) + d - 1;
    const int have = on ? min(x.gt.len[j] - off, L) : 0;
    const int at = have > 0 ? x.gt.start[j] + off : 0;           // (loads from clamped addresses do not wait for each other)
#pragma unroll
    for (int l = 0; l < kAhead; ++l) t[l] = l < 2 || L > 2 ? a.tokens[at + min(l, max(have - 1, 0))] : -1;
    return have;
}
__device__ __forceinline__ void end_string(const Args& a, int have, int (&t)[kAhead]) {
    bool on = true;
#pragma unroll
    for (int l = 0; l < kAhead; ++l) {
        on = on && l < have && t[l] >= 0 && t[l] < a.vocab;      // (a token that cannot be proposed ends the string)
        t[l] = on ? t[l] : -1;
    }
}
__device__ __forceinline__ void fetch_string(const Args& a, const Expand& x, uint32_t place, bool on, int d, int L, int (&t)[kAhead]) {
    const int have = request_string(a, x, place, on, d, L, t);
    end_string(a, have, t);
}
__device__ __forceinline__ void put_string(int* row, const int (&t)[kAhead]) {
    static_assert(kAhead == 8, "two 16-byte words");
    *reinterpret_cast<int4*>(row) = make_int4(t[0], t[1], t[2], t[3]);
    *reinterpret_cast<int4*>(row + 4) = make_int4(t[4], t[5], t[6], t[7]);
}
__device__ __forceinline__ void get_string(const int* row, int (&t)[kAhead]) {
    const int4 lo = *reinterpret_cast<const int4*>(row), hi = *reinterpret_cast<const int4*>(row + 4);
    t[0] = lo.x, t[1] = lo.y, t[2] = lo.z, t[3] = lo.w, t[4] = hi.x, t[5] = hi.y, t[6] = hi.z, t[7] = hi.w;
}
__device__ __forceinline__ bool same_string(const int* row, const int (&t)[kAhead]) {
    int other[kAhead];
    get_string(row, other);
    bool same = true;
#pragma unroll
    for (int l = 0; l < kAhead; ++l) same = same && other[l] == t[l];
    return same;
}
__device__ __forceinline__ uint32_t hash_string(int member, const int (&t)[kAhead]) {
    uint32_t f = static_cast<uint32_t>(member);
#pragma unroll
    for (int l = 0; l < kAhead; ++l) f = (f ^ static_cast<uint32_t>(t[l])) * 0x9e3779b1u, f ^= f >> 15;
    return f * 2654435761u;
}

__device__ __forceinline__ void drop_word(Held& h) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
#pragma unroll
        for (int l = 0; l + 1 < kAhead; ++l) h.t[u][l] = h.t[u][l + 1];
        h.t[u][kAhead - 1] = -1;
    }
}

// The places that this lane's string stands for, of `live` lanes with one each: those that show what the first lane shows
// are all that lane's (0: another lane's, or none).
__device__ __forceinline__ int places_of_lane(int member, const int (&t)[kAhead], bool live) {
    const uint64_t all = __ballot(live);
    if (all == 0) return 0;
    const int lead = __ffsll(static_cast<long long>(all)) - 1;
    bool same = live && member == __builtin_amdgcn_readlane(member, lead);
#pragma unroll
    for (int l = 0; l < kAhead; ++l) same = same && t[l] == __builtin_amdgcn_readlane(t[l], lead);
    const uint64_t equal = __ballot(same);
    return !live ? 0 : (!same ? 1 : (lane_id() == lead ? __popcll(equal) : 0));
}

// One string stays for all places that show the same, with their number as its weight.  A wave's lanes that agree with its first one
// are settled without the table; where hardly any do, nearly all strings differ and the table is left out (1426 places of seven tokens out of eight:
// whole call 29.0 us with it, 23.0 without): false, and the strings stay where they are.
__device__ __forceinline__ bool distinct_strings(Expand& x, Held& h, int n, int threads) {
    const int tid = static_cast<int>(threadIdx.x);
    // a slot of the table: the string that entered it, and 1 << 16 for every place that shows it
    int table = 2 * kFew;
    while (table < 2 * n) table <<= 1;
    const int shift = 32 - __builtin_ctz(static_cast<unsigned>(table));
    for (int i = tid; i < table; i += threads) x.distinct[i] = kEmpty;
    int settled = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const bool live = h.member[u] >= 0;
        h.w[u] = places_of_lane(h.member[u], h.t[u], live);
        settled += __popcll(__ballot(live && h.w[u] == 0));
        if (h.w[u] == 0) h.member[u] = -1;
        if (h.member[u] >= 0) {
            put_string(x.row[tid + u * threads], h.t[u]);
            x.member[tid + u * threads] = static_cast<int8_t>(h.member[u]);
        }
    }
    if (lane_id() == 0) x.red[tid >> 6] = static_cast<uint64_t>(settled);
    __syncthreads();
    settled = 0;
    for (int w = 0; w < threads / 64; ++w) settled += static_cast<int>(x.red[w]);
    if (uniform(settled) < kSettled) return false;
    uint32_t at[kPer], old[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        at[u] = hash_string(h.member[u], h.t[u]) >> shift;
        old[u] = kEmpty;
        if (h.member[u] >= 0) old[u] = atomicCAS(&x.distinct[at[u]], kEmpty, (static_cast<uint32_t>(h.w[u]) << 16) | static_cast<uint32_t>(tid + u * threads));
    }
    bool own[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        own[u] = h.member[u] >= 0;
        if (!own[u]) continue;
        for (int probes = 0; old[u] != kEmpty && probes < table; ++probes) {
            const int j = static_cast<int>(old[u] & 0xffffu);
            if (x.member[j] == h.member[u] && same_string(x.row[j], h.t[u])) {
                atomicAdd(&x.distinct[at[u]], static_cast<uint32_t>(h.w[u]) << 16);
                own[u] = false;
                break;
            }
            at[u] = (at[u] + 1) & (table - 1);
            old[u] = atomicCAS(&x.distinct[at[u]], kEmpty, (static_cast<uint32_t>(h.w[u]) << 16) | static_cast<uint32_t>(tid + u * threads));
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (own[u]) h.w[u] = static_cast<int>(x.distinct[at[u]] >> 16);
        h.member[u] = own[u] ? h.member[u] : -1;
    }
    return true;
}

// Threads that n strings are for, of those that are left.
__device__ __forceinline__ int threads_for(int n, int threads) {
    return n <= 64 ? 64 : min(threads, n <= kFew ? kFewThreads : (n <= 2 * kFew ? 2 * kFewThreads : kThreads));
}

// The strings that are left move to the first threads; the waves without any end.  Returns their number.
__device__ __forceinline__ int pack_strings(Expand& x, Held& h, int& threads) {
    const int tid = static_cast<int>(threadIdx.x);
    if (tid == 0) x.n_held = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int at = wave_append(&x.n_held, h.member[u] >= 0);
        if (h.member[u] >= 0) {
            put_string(x.row[at], h.t[u]);
            x.id[at] = static_cast<uint16_t>(h.id[u]), x.weight[at] = static_cast<uint16_t>(h.w[u]);
            x.member[at] = static_cast<int8_t>(h.member[u]);
        }
    }
    __syncthreads();
    const int n = uniform(x.n_held);
    threads = threads_for(n, threads);
    if (tid >= threads) __builtin_amdgcn_endpgm();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int at = tid + u * threads;
        h.member[u] = -1;
        if (at >= n) continue;
        get_string(x.row[at], h.t[u]);
        h.id[u] = x.id[at], h.w[u] = x.weight[at], h.member[u] = x.member[at];
    }
    __syncthreads();                                             // the tables lie where the strings were
    return n;
}

// The distinct strings, of at most kAhead words, of the n places on a list in global memory, which belong to the root: in
// the first threads, which alone go on.  Returns their number; -1, with all threads, if there are more than kSmall.
__device__ __forceinline__ int distinct_listed(const Args& a, Expand& x, const uint32_t* list, int n, int L, Held& h, int& threads) {
    const int tid = static_cast<int>(threadIdx.x);
    constexpr int kTable = 2 * kSmall, kShift = 32 - __builtin_ctz(static_cast<unsigned>(kTable));
    // a slot of the table: 1 << 16 for every place that shows the string, which is x.fresh[slot] of this round
    // or x.kept[slot - kThreads] of an earlier one
    for (int i = tid; i < kTable; i += kThreads) x.distinct[i] = kEmpty;
    if (tid == 0) x.n_held = 0;
    __syncthreads();                                             // (the last level's list is written)
    uint32_t place = list[min(tid, n - 1)];
    int got[kAhead], have = request_string(a, x, place, tid < n, 1, L, got);
    for (int i0 = 0; i0 < n; i0 += kThreads) {
        // (the next round's places are requested in front of this round's strings, its strings behind them)
        place = list[min(i0 + kThreads + tid, n - 1)];
        int t[kAhead];
#pragma unroll
        for (int l = 0; l < kAhead; ++l) t[l] = got[l];
        end_string(a, have, t);
        const int places = places_of_lane(0, t, t[0] >= 0);
        bool own = places > 0;
        if (own) put_string(x.fresh[tid], t);
        have = request_string(a, x, place, i0 + kThreads + tid < n, 1, L, got);
        __syncthreads();
        const int so_far = uniform(x.n_held);
        if (so_far > kSmall || (i0 == kThreads && so_far * n > kThreads * kHopeless)) return -1;
        uint32_t at = hash_string(0, t) >> kShift;
        if (own) {
            const uint32_t enter = (static_cast<uint32_t>(places) << 16) | static_cast<uint32_t>(tid);
            uint32_t old = atomicCAS(&x.distinct[at], kEmpty, enter);
            for (int probes = 0; old != kEmpty && probes < kTable; ++probes) {
                const int j = static_cast<int>(old & 0xffffu);
                if (same_string(j < kThreads ? x.fresh[j] : x.kept[j - kThreads], t)) {
                    atomicAdd(&x.distinct[at], static_cast<uint32_t>(places) << 16);
                    own = false;
                    break;
                }
                at = (at + 1) & (kTable - 1);
                old = atomicCAS(&x.distinct[at], kEmpty, enter);
            }
        }
        __syncthreads();
        const int k = wave_append(&x.n_held, own);
        if (own && k < kSmall) {
            put_string(x.kept[k], t);
            x.list[k] = static_cast<uint16_t>(at);
            x.distinct[at] += static_cast<uint32_t>(kThreads + k - tid);
        }
    }
    __syncthreads();
    const int n_str = uniform(x.n_held);
    if (n_str > kSmall) return -1;
    threads = threads_for(n_str, threads);
    if (tid >= threads) __builtin_amdgcn_endpgm();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = tid + u * threads;
        h.id[u] = e, h.w[u] = 0, h.member[u] = -1;
        if (e >= n_str) continue;
        get_string(x.kept[e], h.t[u]);
        h.w[u] = static_cast<int>(x.distinct[x.list[e]] >> 16), h.member[u] = 0;
    }
    __syncthreads();                                             // the tables lie where the strings were
    return n_str;
}

// `n` places show the pair: its entry, and whether it was new.
__device__ __forceinline__ int enter_pair(uint64_t* table, int slots, uint32_t pair, int n, bool* entered) {
    const uint64_t count = (1ull << 48) | (static_cast<uint64_t>(static_cast<uint32_t>(n)) << 32);
    int at = static_cast<int>((pair * 2654435761u) >> (32 - __builtin_ctz(static_cast<unsigned>(slots))));
    for (int probes = 0; probes < slots; ++probes) {             // (fewer pairs than slots: it always ends before)
        uint64_t word = table[at];
        if (word == kNoPair) {
            word = atomicCAS(reinterpret_cast<unsigned long long*>(&table[at]), kNoPair, pair | count);
            if (word == kNoPair) {
                *entered = true;
                break;
            }
        }
        if (static_cast<uint32_t>(word) == pair) {
            atomicAdd(reinterpret_cast<unsigned long long*>(&table[at]), count);
            break;
        }
        at = (at + 1) & (slots - 1);
    }
    return at;
}

// One wave: ranks of the up to 64 candidates (one per lane, 0 = none; all differ), kMaxTopK or more for the others.
__device__ __forceinline__ int rank_lanes(uint64_t v, uint64_t mask, int n_pick) {
    const int n_cand = __popcll(mask);
    int rank = v != 0 ? 0 : kMaxTopK;
    if (n_cand <= kRankWave) {
        if (n_cand > 1)
            for (uint64_t left = mask; left != 0; left &= left - 1)
                rank += lane_value(v, __ffsll(static_cast<long long>(left)) - 1) > v ? 1 : 0;
    } else {
        uint64_t rest = v;
        rank = kMaxTopK;
        for (int round = 0; round < n_pick; ++round) {
            const uint64_t best = wave_max_u64(rest);
            if (rest == best) rank = round, rest = 0;
        }
    }
    return rank;
}

// An entry of the table as a candidate of the beam: count << 32 | ~pair, 0 if fewer than `least` places show it.
__device__ __forceinline__ uint64_t candidate(uint64_t word, int least) {
    const uint32_t count = static_cast<uint32_t>(word >> 32) & 0xffffu;
    return static_cast<int>(count) >= least ? (static_cast<uint64_t>(count) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(word)) : 0;
}

// One wave: the picks of level d among the level's pairs become draft nodes.  Returns the strings that go on.
__device__ __forceinline__ int pick_listed(const Args& a, Expand& x, int buf, int d, int least) {
    const int lane = lane_id(), n_pairs = uniform(x.n_list[buf]);
    if (n_pairs <= 64) {
        const int at = lane < n_pairs ? x.list[lane] : 0;
        const uint64_t word = x.pair[buf][at];
        const uint64_t v = lane < n_pairs ? candidate(word, least) : 0;
        const uint64_t mask = __ballot(v != 0);
        const int n_pick = min(__popcll(mask), a.top_k), rank = rank_lanes(v, mask, n_pick);
        if (rank < n_pick) {
            x.rank[buf][at] = static_cast<int8_t>(rank);
            put_node(x, d, a.top_k, rank, v);
        }
        return wave_sum(rank < n_pick ? static_cast<int>(word >> 48) : 0);
    }
    // a longer list: lane j keeps the j-th best so far
    uint64_t kept = 0;
    int kept_at = 0, n_cand = 0;
    for (int i0 = 0; i0 < n_pairs; i0 += kListed * 64) {
        uint64_t v[kListed + 1];
        int at[kListed + 1];
#pragma unroll
        for (int u = 0; u < kListed; ++u) at[u] = x.list[min(i0 + u * 64 + lane, n_pairs - 1)];
#pragma unroll
        for (int u = 0; u < kListed; ++u) {
            v[u] = candidate(x.pair[buf][at[u]], least);
            if (i0 + u * 64 + lane >= n_pairs) v[u] = 0;
            n_cand += __popcll(__ballot(v[u] != 0));
        }
        v[kListed] = kept, at[kListed] = kept_at;
        kept = 0;
        const int rounds = min(n_cand, a.top_k);
        for (int round = 0; round < rounds; ++round) {
            uint64_t best = 0;
            int of = 0;
#pragma unroll
            for (int u = 0; u <= kListed; ++u)
                if (v[u] > best) best = v[u], of = at[u];
            const uint64_t top = wave_max_u64(best);
            of = __builtin_amdgcn_readlane(of, __ffsll(static_cast<long long>(__ballot(best == top))) - 1);
#pragma unroll
            for (int u = 0; u <= kListed; ++u)
                if (v[u] == top) v[u] = 0;
            if (lane == round) kept = top, kept_at = of;
        }
    }
    const int n_pick = min(n_cand, a.top_k);
    if (lane < n_pick) {
        x.rank[buf][kept_at] = static_cast<int8_t>(lane);
        put_node(x, d, a.top_k, lane, kept);
    }
    return wave_sum(lane < n_pick ? static_cast<int>(x.pair[buf][kept_at] >> 48) : 0);
}

__device__ __forceinline__ void clear_pairs(Expand& x, int buf, int slots, int from, int step) {
    for (int i = 2 * from; i < slots; i += 2 * step)
        *reinterpret_cast<ulonglong2*>(&x.pair[buf][i]) = make_ulonglong2(kNoPair, kNoPair);
    if (from == 0) x.n_list[buf] = 0;
}

// Levels from d on, over the first words of the n strings, until no more than `most` strings are left or `levels` levels are
// done; n = strings left, 0 if the search has ended.  Returns the levels done.
__device__ __forceinline__ int count_levels(const Args& a, Expand& x, Held& h, int d, int levels, int threads, int least,
                                            int most, int& n) {
    const int tid = static_cast<int>(threadIdx.x);
    int slots = 256, done = 0, buf = 0;
    while (slots < kSlots && slots < 4 * n) slots <<= 1;
    clear_pairs(x, 0, slots, tid, threads);
    __syncthreads();
    for (; done < levels && n > most; ++done, ++d, buf ^= 1) {
        int at[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const bool go = h.member[u] >= 0 && h.t[u][0] >= 0;
            bool entered = false;
            at[u] = -1;
            if (go)
                at[u] = enter_pair(x.pair[buf], slots, (static_cast<uint32_t>(h.member[u]) << 24) | static_cast<uint32_t>(h.t[u][0]), h.w[u], &entered);
            const int to = wave_append(&x.n_list[buf], entered);
            if (entered) x.list[to] = static_cast<uint16_t>(at[u]), x.rank[buf][at[u]] = -1;
        }
        drop_word(h);
        __syncthreads();
        if (tid < 64) {
            const int left = pick_listed(a, x, buf, d, least);
            if (tid == 0) x.n_left = left;
        } else {
            clear_pairs(x, buf ^ 1, slots, tid - 64, threads - 64);
        }
        __syncthreads();
        n = uniform(x.n_left);
#pragma unroll
        for (int u = 0; u < kPer; ++u) h.member[u] = at[u] >= 0 ? x.rank[buf][at[u]] : -1;
    }
    return done;
}

// One wave, one string per lane: `levels` levels from d on; false if the search has ended.
__device__ __forceinline__ bool search_lanes(const Args& a, Expand& x, Held& h, int d, int levels, int least) {
    const int lane = lane_id(), w = h.w[0], top_k = a.top_k;
    const bool single = __ballot(h.member[0] >= 0 && w > 1) == 0;
    int member = h.member[0];
    // lane r: the ancestors of the member of rank r
    uint64_t ancestors = x.msk[lane < top_k ? member_slot(d, top_k, lane) : 0];
    for (int p = 0; p < levels; ++p, ++d) {
        const int token = h.t[0][0], slot0 = 1 + (d - 1) * top_k;
        drop_word(h);
        const bool go = member >= 0 && token >= 0;
        const uint32_t pair = (static_cast<uint32_t>(member) << 24) | static_cast<uint32_t>(token);
        const uint64_t all = __ballot(go);
        if (all == 0) return false;
        int lead = __ffsll(static_cast<long long>(all)) - 1;
        uint32_t shown = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(pair), lead));
        uint64_t same = __ballot(go && pair == shown);
        if (same == all) {
            // all show the same: nothing to rank
            const int count = single ? __popcll(all) : wave_sum(go ? w : 0);
            if (count < least) return false;
            const int r = static_cast<int>(shown >> 24);
            ancestors = (1ull << slot0) | lane_value(ancestors, r);
            if (lane == 0)
                x.tok[slot0] = static_cast<int>(shown & 0xffffffu), x.par[slot0] = member_slot(d, top_k, r), x.num[slot0] = count, x.msk[slot0] = ancestors;
            member = go ? 0 : -1;
            continue;
        }
        int v_hi = 0, v_lo = 0;
        uint64_t left = all;
        const auto settle = [&]() __attribute__((always_inline)) {          // the lanes that show what `lead` shows
            const int count = single ? __popcll(same) : wave_sum((same >> lane) & 1 ? w : 0);
            left &= ~same;
            const int hi = count >= least ? count : 0;
            v_hi = lane == lead ? hi : v_hi, v_lo = lane == lead ? static_cast<int>(~shown) : v_lo;
        };
        settle();
        int peeled = 1;
        while (left != 0) {
            if (peeled < kPeel) {
                lead = __ffsll(static_cast<long long>(left)) - 1;
                shown = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(pair), lead));
                same = __ballot(pair == shown) & left;
                settle();
                ++peeled;
                continue;
            }
            // Many pairs: a lane that hashes to the same word as others and finds its own pair there counts with the
            // one that wrote it.  (The next round takes those whose word another pair took.)
            const bool open = (left >> lane) & 1;
            uint32_t* const word = reinterpret_cast<uint32_t*>(x.list) + ((pair * 2654435761u) >> (32 - kMeetLog2));
            uint32_t* const met = x.distinct;
            met[lane] = 0;
            if (open) *word = static_cast<uint32_t>(lane);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int at = open ? static_cast<int>(*word) : lane;
            const bool joins = static_cast<uint32_t>(__shfl(static_cast<int>(pair), at, 64)) == pair && open;
            if (joins) atomicAdd(&met[at], static_cast<uint32_t>(w));
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int count = static_cast<int>(met[lane]);
            if (count > 0) v_hi = count >= least ? count : 0, v_lo = static_cast<int>(~pair);
            left &= ~__ballot(joins);
            peeled = 0;
        }
        const uint64_t v = v_hi > 0 ? (static_cast<uint64_t>(static_cast<uint32_t>(v_hi)) << 32) | static_cast<uint32_t>(v_lo) : 0;
        const uint64_t mask = __ballot(v_hi > 0);
        const int n_pick = min(__popcll(mask), top_k);
        if (n_pick == 0) return false;
        const int rank = rank_lanes(v, mask, n_pick);
        int now = -1, tok = 0, par = 0, num = 0;
        uint64_t msk = 0;
        for (int r = 0; r < n_pick; ++r) {
            const int of = __ffsll(static_cast<long long>(__ballot(rank == r))) - 1;
            const uint64_t pick = lane_value(v, of);
            shown = ~static_cast<uint32_t>(pick);
            const int up = static_cast<int>(shown >> 24);
            const uint64_t m = (1ull << (slot0 + r)) | lane_value(ancestors, up);
            now = go && pair == shown ? r : now;
            const bool here = lane == r;
            tok = here ? static_cast<int>(shown & 0xffffffu) : tok, par = here ? member_slot(d, top_k, up) : par;
            num = here ? static_cast<int>(pick >> 32) : num, msk = here ? m : msk;
        }
        member = now;
        if (lane < n_pick) x.tok[slot0 + lane] = tok, x.par[slot0 + lane] = par, x.num[slot0 + lane] = num, x.msk[slot0 + lane] = msk;
        ancestors = msk;
    }
    h.member[0] = member;
    return true;
}

// L levels from level d on, over the first L words of the n_str strings that `threads` threads hold; threads that are no
// longer needed end.  `last`: no levels come behind them, so equal strings need no place each.  True if the search has ended.
__device__ __forceinline__ bool search_strings(const Args& a, Expand& x, Held& h, int d, int L, bool last, int least, int n_str, int& threads) {
    const int tid = static_cast<int>(threadIdx.x);
    int lvl = 0;
    bool ended = n_str == 0;
    if (n_str > 64) {
        // the levels on which all strings agree, for one member, as a string of the first wave shows them (one that goes on to the
        // last, if there is one), and the places that show that string
        bool holder = false;
        if (tid < 64) {
            bool full = h.member[0] >= 0;
#pragma unroll
            for (int l = 0; l < kAhead; ++l) full = full && (l >= L || h.t[0][l] >= 0);
            const uint64_t ready = __ballot(full);
            holder = tid == (ready != 0 ? __ffsll(static_cast<long long>(ready)) - 1 : 0);
            if (holder) {
#pragma unroll
                for (int l = 0; l < kAhead; ++l) x.lead[l] = h.t[0][l];
                x.lead_member = h.member[0], x.common = L, x.n_on = 0;
            }
        }
        __syncthreads();
        const int member = uniform(x.lead_member);
        int all = member >= 0 ? L : 0;
        bool same[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) same[u] = h.member[u] >= 0 && h.member[u] == member;
#pragma unroll
        for (int l = kAhead - 1; l >= 0; --l) {
            const int lead = x.lead[l];
            bool parts = lead < 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const bool equal = h.t[u][l] == lead;
                parts = parts || (h.member[u] >= 0 && (h.member[u] != member || !equal));
                same[u] = same[u] && equal;
            }
            if (l < all && __ballot(parts) != 0) all = l;
        }
        uint32_t n_on = 0;                                       // places: those that show the string << 16 | all
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            n_on += (h.member[u] >= 0 ? static_cast<uint32_t>(h.w[u]) : 0u) + (same[u] ? static_cast<uint32_t>(h.w[u]) << 16 : 0u);
        n_on = static_cast<uint32_t>(wave_sum(static_cast<int>(n_on)));
        if (lane_id() == 0) {
            atomicMin(&x.common, all);
            atomicAdd(&x.n_on, n_on);
        }
        __syncthreads();
        lvl = uniform(x.common);
        const int count = uniform(static_cast<int>(x.n_on & 0xffffu)), n_same = uniform(static_cast<int>(x.n_on >> 16));
        if (lvl > 0) {
            if (count < least) ended = true;
            if (!ended && tid == 0)
                for (int l = 0; l < lvl; ++l)
                    put_node(x, d + l, a.top_k, 0,
                             (static_cast<uint64_t>(static_cast<uint32_t>(count)) << 32) |
                                 static_cast<uint32_t>(~((static_cast<uint32_t>(l == 0 ? member : 0) << 24) | static_cast<uint32_t>(x.lead[l]))));
#pragma unroll
            for (int u = 0; u < kPer; ++u) h.member[u] = min(h.member[u], 0);
            for (int l = 0; l < lvl; ++l) drop_word(h);
        }
        // a string that half of the places show, or whose repeats are what is more than one wave's work, stays once
        if (last && !ended && lvl < L && n_same > 1 && (2 * n_same >= count || n_str - n_same < 64)) {
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (same[u] && !(holder && u == 0)) h.member[u] = -1;
            if (holder) h.w[0] = n_same;
            n_str = pack_strings(x, h, threads);
        }
        while (!ended && lvl < L && n_str > 64) {
            lvl += count_levels(a, x, h, d + lvl, L - lvl, threads, least, threads > kFewThreads ? kPer / 2 * threads : 64, n_str);
            ended = n_str == 0;
            if (!ended && lvl < L) n_str = pack_strings(x, h, threads);
        }
    }
    if (!ended && lvl < L) ended = !search_lanes(a, x, h, d + lvl, L - lvl, least);
    return ended;
}

// Levels d .. levels over the n places in x.place / x.owner, by the whole workgroup.
__device__ __forceinline__ void search_places(const Args& a, Expand& x, int d, int levels, int least, int n) {
    const int tid = static_cast<int>(threadIdx.x);
    int threads = kThreads;
    while (d <= levels) {
        threads = threads_for(n, threads);
        if (tid >= threads) __builtin_amdgcn_endpgm();
        const int L = min(levels - d + 1, kAhead);
        Held h;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + u * threads;
            const uint32_t place = i < n ? x.place[i] : 0u;
            const int own = i < n ? x.owner[i] : -1;
            fetch_string(a, x, place, own >= 0, d, L, h.t[u]);
            h.id[u] = i, h.w[u] = 1, h.member[u] = h.t[u][0] >= 0 ? own : -1;
        }
        int n_str = n;
        if (n > kFew && d + L > levels && L >= kDistinctLevels && distinct_strings(x, h, n, threads)) n_str = pack_strings(x, h, threads);
        const bool ended = search_strings(a, x, h, d, L, d + L > levels, least, n_str, threads);
        d += L;
        if (ended || d > levels) break;
        // the places that go on, in front (each string is one place: distinct strings are for the last round)
        uint32_t place[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) place[u] = h.member[u] >= 0 ? x.place[h.id[u]] : 0u;
        if (tid == 0) x.n_held = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int at = wave_append(&x.n_held, h.member[u] >= 0);
            if (h.member[u] >= 0) x.place[at] = place[u], x.owner[at] = static_cast<int8_t>(h.member[u]);
        }
        __syncthreads();
        n = uniform(x.n_held);
    }
}

__global__ __launch_bounds__(kThreads) void draft_expand_kernel(Args a) {
    __shared__ Expand x;
    const int b = blockIdx.x, tid = threadIdx.x;
    const int T = 1 + a.top_k * a.gamma_max;
    const int plen = min(max(a.pattern_len[b], 0), a.p_max);
    const int want = a.max_spec_tokens[b];
    // What has to be known first, each part by a wave of its own, one barrier behind all: the longest match over the stretches
    // and how many of its places come before part p (at most kMaxParts = 256 parts: four per lane); the group's table; the empty
    // draft.  (One after the other, with eleven barriers of sixteen waves, it took 2 .. 3 us longer: with the match kernel's start
    // the whole call 37.6 -> 35.0 us on 16 chains, 121.6 -> 119.2 us on the multi-path batch.)
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    if (wave == 0) {
        int2 h[kMaxParts / 64];
#pragma unroll
        for (int k = 0; k < kMaxParts / 64; ++k) {
            const int p = tid * (kMaxParts / 64) + k;
            h[k] = p < a.parts ? a.part_hdr[static_cast<size_t>(b) * a.parts + p] : make_int2(0, 0);
        }
        int best = 0;
#pragma unroll
        for (int k = 0; k < kMaxParts / 64; ++k)
            if (h[k].x > 0) best = max(best, h[k].y);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
        int c[kMaxParts / 64], sum = 0;
#pragma unroll
        for (int k = 0; k < kMaxParts / 64; ++k) {
            c[k] = h[k].y == best ? h[k].x : 0;
            sum += c[k];
        }
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (tid >= o) incl += up;
        }
        int before = incl - sum;
#pragma unroll
        for (int k = 0; k < kMaxParts / 64; ++k) {
            x.first[tid * (kMaxParts / 64) + k] = before;
            before += c[k];
        }
        if (tid == 63) x.first[kMaxParts] = before;
        if (tid == 0) x.n = 0, x.best_len = best;
    } else if (wave == 1) {
        load_group(a, a.req_group[b], x.gt);
    } else if (wave == 2 && tid - 128 < T) {
        const int t = tid - 128;
        x.tok[t] = t == 0 && plen > 0 ? a.pattern[static_cast<size_t>(b) * a.p_max + a.p_max - 1] : -1;
        x.par[t] = t == 0 ? -1 : -2;
        x.num[t] = 0;
        x.msk[t] = 1ull << t;
    }
    __syncthreads();
    if (x.gt.bad && tid == 0 && a.status) atomicOr(a.status, x.gt.bad);
    const int p_star = x.gt.n_seq > 0 ? x.best_len : 0;
    const int n_kept = p_star > 0 ? x.first[a.parts] : 0;        // >= the places of the longest match
    const auto put_draft = [&]() {
        if (tid < T) {
            const size_t o = static_cast<size_t>(b) * T + tid;
            a.draft_tokens[o] = x.tok[tid];
            a.tree_parent[o] = x.par[tid];
            a.tree_mask[o] = x.msk[tid];
            if (a.node_count) a.node_count[o] = x.num[tid];
        }
        if (tid == 0 && a.match_len) a.match_len[b] = p_star;
    };
    if (uniform(n_kept) == 0) {                                  // no match: the empty draft
        put_draft();
        return;
    }
    uint32_t* cur = a.list_b + static_cast<size_t>(b) * a.cap;
    uint32_t* nxt = a.list_a + static_cast<size_t>(b) * a.cap;
    bool handed_over = n_kept <= kSmall;
    for (int i0 = 0; i0 < n_kept; i0 += kThreads) {
        const int i = i0 + tid;
        uint32_t pl = 0;
        if (i < n_kept) {
            int lo = 0, hi = a.parts;                              // the part that holds kept place i
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (x.first[mid] <= i) lo = mid; else hi = mid;
            }
            pl = nxt[static_cast<size_t>(lo) * a.chunk + (i - x.first[lo])];
        }
        const bool hit = i < n_kept && place_len(pl) == p_star;
        const int at = wave_append(&x.n, hit);
        if (hit) {
            if (handed_over)
                x.place[at] = pl, x.owner[at] = 0;
            else
                cur[at] = pl;
        }
    }
    __syncthreads();
    const int n_root = x.n;
    const int levels = p_star > 0 ? min(max(want, 0), a.gamma_max) : 0;
    const float threshold = a.min_confidence * static_cast<float>(n_root);
    if (tid == 0) {
        x.num[0] = n_root;
        x.mem[0] = Member{0, n_root, 0};
        x.nmem = 1;
    }
    __syncthreads();

    int d = 1;
    const int least = uniform(static_cast<int>(ceilf(threshold)));       // (counts are below 2^24: the same test)
    bool done = false;
    if (!handed_over && n_root > kSmall && n_root < kManyPlaces && levels >= kDistinctLevels && levels <= kAhead) {
        Held h;
        int threads = kThreads;
        const int n_str = distinct_listed(a, x, cur, uniform(n_root), uniform(levels), h, threads);
        if (n_str >= 0) {
            search_strings(a, x, h, 1, uniform(levels), true, least, n_str, threads);
            done = true;
        }
    }
    // ---- places in global memory: as long as a level holds more than kSmall places ----
    for (; d <= levels && !handed_over && !done; ++d) {
        const int nmem = x.nmem;
        const int n_level = x.mem[nmem - 1].base + x.mem[nmem - 1].n;
        if (n_level <= kSmall) {
            for (int e = tid; e < n_level; e += kThreads) {
                int r = 0;
                while (r + 1 < nmem && e >= x.mem[r + 1].base) ++r;
                x.place[e] = cur[e], x.owner[e] = static_cast<int8_t>(r);
            }
            handed_over = true;
            __syncthreads();
            break;
        }
        // The tokens that four places per thread show at this level, with the rank of the member that owns
        // each place, as keys.  The four places are requested together, then the four tokens (from addresses
        // clamped into the pool), so that a thread waits twice per round, not eight times.
        auto keys_of = [&](int e0, uint32_t (&pl)[4], uint32_t (&key)[4], bool (&outside)[4]) {
            int at[4];
            bool ok[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) pl[u] = cur[min(e0 + u * kThreads + tid, n_level - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = place_seq(pl[u]), off = place_off(pl[u]) + d - 1;
                ok[u] = e0 + u * kThreads + tid < n_level && off < x.gt.len[j];
                at[u] = ok[u] ? x.gt.start[j] + off : 0;
            }
            int t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = a.tokens[at[u]];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * kThreads + tid;
                int r = 0;
                while (r + 1 < nmem && e >= x.mem[r + 1].base) ++r;
                outside[u] = ok[u] && (t[u] < 0 || t[u] >= a.vocab);       // a token that cannot be proposed
                key[u] = ok[u] && !outside[u] ? (static_cast<uint32_t>(r) << 24) | static_cast<uint32_t>(t[u]) : kEmpty;
            }
        };
        // A level of up to 8 places per thread is fetched once (two dependent round trips) and kept in registers
        // for the three passes below (agreement, counting, reassignment); longer levels are fetched pass by pass.
        constexpr int kHeld = 8;
        const bool held = n_level <= kHeld * kThreads;
        uint32_t hpl[kHeld], hkey[kHeld];
        bool hout[kHeld];
        if (held) {
            keys_of(0, *reinterpret_cast<uint32_t(*)[4]>(&hpl[0]), *reinterpret_cast<uint32_t(*)[4]>(&hkey[0]),
                    *reinterpret_cast<bool(*)[4]>(&hout[0]));
            keys_of(4 * kThreads, *reinterpret_cast<uint32_t(*)[4]>(&hpl[4]), *reinterpret_cast<uint32_t(*)[4]>(&hkey[4]),
                    *reinterpret_cast<bool(*)[4]>(&hout[4]));
        }
        // f(round, places, keys, outside) for every round of four places per thread
        auto for_each_round = [&](auto&& f) {
            if (held) {
                f(0, *reinterpret_cast<uint32_t(*)[4]>(&hpl[0]), *reinterpret_cast<uint32_t(*)[4]>(&hkey[0]),
                  *reinterpret_cast<bool(*)[4]>(&hout[0]));
                if (n_level > 4 * kThreads)
                    f(1, *reinterpret_cast<uint32_t(*)[4]>(&hpl[4]), *reinterpret_cast<uint32_t(*)[4]>(&hkey[4]),
                      *reinterpret_cast<bool(*)[4]>(&hout[4]));
            } else {
                for (int e0 = 0; e0 < n_level; e0 += 4 * kThreads) {
                    uint32_t pl[4], key[4];
                    bool outside[4];
                    keys_of(e0, pl, key, outside);
                    f(e0 / (4 * kThreads), pl, key, outside);
                }
            }
        };
        // A single member whose places all show the same token (inside a phrase that recurs): one pass finds
        // that out and counts them; the place list stays as it is (places whose sequence ended stay ended).
        if (nmem == 1) {
            if (tid == 0) x.ref[0] = -1, x.ref_cnt[0] = 0;
            __syncthreads();
            bool agree = true;
            int wave_count = 0;
            for_each_round([&](int round, uint32_t (&pl)[4], uint32_t (&key)[4], bool (&outside)[4]) {
                if (round == 0) {                  // any token of the first round serves as the reference
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (key[u] != kEmpty) x.ref[0] = static_cast<int>(key[u] & 0xffffffu);
                    __syncthreads();
                }
                const int ref = x.ref[0];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (outside[u]) agree = false;
                    if (key[u] != kEmpty && static_cast<int>(key[u] & 0xffffffu) != ref) agree = false;
                    wave_count += __popcll(__ballot(key[u] != kEmpty));
                }
            });
            if (lane_id() == 0 && wave_count) atomicAdd(&x.ref_cnt[0], wave_count);
            if (__syncthreads_and(agree ? 1 : 0)) {
                const int c = x.ref_cnt[0];
                if (c == 0 || static_cast<float>(c) < threshold) {
                    d = levels + 1;
                    break;
                }
                if (tid == 0) {
                    x.pick[0] = (static_cast<uint64_t>(c) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(x.ref[0]));
                    emit_nodes(x, d, a.top_k, 1);
                    x.mem[0] = Member{0, n_level, x.next[0].slot};
                }
                __syncthreads();
                continue;
            }
        }
        int n_pick = 0;
        // Pass 0 counts in a hash table.  Only if more distinct (member, token) pairs turn up than the
        // table has slots do further passes count token ranges in a directly indexed table.
        const int range = kTableSlots / nmem;                     // tokens per member in a ranged pass
        const int n_pass_ranged = (a.vocab + range - 1) / range;
        const int shift = 32 - __builtin_ctz(static_cast<unsigned>(kTableSlots));
        for (int pass = 0; pass <= n_pass_ranged; ++pass) {
            const bool hashed = pass == 0;
            for (int s = tid; s < kTableSlots; s += kThreads) x.key[s] = kEmpty, x.cnt[s] = 0;
            if (tid == 0) x.overflow = 0;
            __syncthreads();
            const int lo_tok = (pass - 1) * range;
            for_each_round([&](int, uint32_t (&pl)[4], uint32_t (&key)[4], bool (&outside)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (hashed) {
                        if (key[u] != kEmpty) hash_add(x, kTableSlots, shift, key[u], 1u);
                    } else if (key[u] != kEmpty) {
                        const int t = static_cast<int>(key[u] & 0xffffffu) - lo_tok;
                        if (t >= 0 && t < range) {
                            const int s = static_cast<int>(key[u] >> 24) * range + t;
                            x.key[s] = key[u];
                            atomicAdd(&x.cnt[s], 1u);
                        }
                    }
                }
            });
            __syncthreads();
            const bool overflow = x.overflow != 0;
            if (!(hashed && overflow)) n_pick = pick_top(x, kTableSlots, threshold, a.top_k, n_pick);
            if (hashed && !overflow) break;
        }
        if (n_pick == 0) {
            d = levels + 1;
            break;
        }
        if (tid == 0) emit_nodes(x, d, a.top_k, n_pick);
        __syncthreads();
        if (d < levels) {
            for_each_round([&](int, uint32_t (&pl)[4], uint32_t (&key)[4], bool (&outside)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    int child = -1;
                    if (key[u] != kEmpty)
                        for (int j = 0; j < n_pick; ++j)
                            if (~static_cast<uint32_t>(x.pick[j]) == key[u]) child = j;
                    // one member's places mostly go to one child: append wave by wave, child by child
                    for (int j = 0; j < n_pick; ++j) {
                        if (__ballot(child == j) == 0) continue;
                        const int at = wave_append(&x.fill[j], child == j);
                        if (child == j) nxt[x.next[j].base + at] = pl[u];
                    }
                }
            });
        }
        __syncthreads();
        if (tid < n_pick) x.mem[tid] = x.next[tid];
        if (tid == 0) x.nmem = n_pick;
        uint32_t* t = cur;
        cur = nxt;
        nxt = t;
        __syncthreads();
    }

    // ---- few enough places: strings ----
    if (handed_over && !done && d <= levels) {
        const int n_places = min(x.mem[x.nmem - 1].base + x.mem[x.nmem - 1].n, kSmall);
        search_places(a, x, uniform(d), uniform(levels), least, uniform(n_places));
    }
    __syncthreads();

    put_draft();
}

}  // namespace draft
}  // namespace seer

namespace {

struct DraftShape {
    int parts, chunk, cap;
    size_t off_hdr, off_a, off_b, total;
};

int draft_shape(const seer_draft_params* p, DraftShape* s) {
    using namespace seer::draft;
    if (!p || p->B < 0 || p->n_groups < 1 || p->n_seq < 1 || p->pool_tokens < 4 || p->max_group_tokens < 1) return SEER_EINVAL;
    if (p->gamma_max < 1 || p->top_k < 1 || p->pattern_lookup_max < 1 || p->pattern_lookup_min < 0 || p->vocab < 1)
        return SEER_EINVAL;
    if (!(p->min_confidence >= 0.0f) || !(p->min_confidence <= 1.0f)) return SEER_EINVAL;
    if (p->pattern_lookup_min > p->pattern_lookup_max) return SEER_ESHAPE;
    if (1 + static_cast<int64_t>(p->top_k) * p->gamma_max > SEER_MAX_T) return SEER_ESHAPE;
    if (p->top_k > kMaxTopK || p->pattern_lookup_max > kMaxPattern || p->vocab > (1 << 24) ||
        p->pool_tokens > 0x7fff0000ll || p->n_groups > 65535)
        return SEER_EUNSUPPORTED;
    int parts = (p->max_group_tokens + kTokensPerPart - 1) / kTokensPerPart;
    parts = parts < 1 ? 1 : (parts > kMaxParts ? kMaxParts : parts);
    int chunk = (p->max_group_tokens + parts - 1) / parts;
    chunk = (chunk + 3) & ~3;
    s->parts = parts, s->chunk = chunk, s->cap = parts * chunk;
    auto up = [](size_t v) { return (v + 255) & ~static_cast<size_t>(255); };
    const size_t B = static_cast<size_t>(p->B > 0 ? p->B : 1);
    s->off_hdr = 0;
    s->off_a = up(B * parts * sizeof(int2));
    s->off_b = s->off_a + up(B * s->cap * sizeof(uint32_t));
    s->total = s->off_b + up(B * s->cap * sizeof(uint32_t));
    return SEER_OK;
}

}  // namespace

extern "C" size_t seer_draft_workspace(const seer_draft_params* p) {
    DraftShape s;
    return draft_shape(p, &s) == SEER_OK ? s.total : 0;
}

extern "C" int seer_draft(const int32_t* tokens, const int32_t* seq_start, const int32_t* seq_len,
                          const int32_t* group_first, const int32_t* req_group, const int32_t* pattern,
                          const int32_t* pattern_len, const int32_t* max_spec_tokens, const seer_draft_params* p,
                          int32_t* draft_tokens, int32_t* tree_parent, uint64_t* tree_mask, int32_t* node_count,
                          int32_t* match_len, int32_t* status, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
    DraftShape s;
    const int shape_rc = draft_shape(p, &s);
    if (shape_rc != SEER_OK) return shape_rc;
    if (p->B == 0) return SEER_OK;
    if (!tokens || !seq_start || !seq_len || !group_first || !req_group || !pattern || !pattern_len || !max_spec_tokens ||
        !draft_tokens || !tree_parent || !tree_mask)
        return SEER_EINVAL;
    if (!workspace || workspace_bytes < s.total) return SEER_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) % 16 != 0 || reinterpret_cast<uintptr_t>(tokens) % 16 != 0) return SEER_EALIGN;
    seer::draft::Args a{};
    a.tokens = tokens, a.seq_start = seq_start, a.seq_len = seq_len, a.group_first = group_first;
    a.req_group = req_group, a.pattern = pattern, a.pattern_len = pattern_len, a.max_spec_tokens = max_spec_tokens;
    a.draft_tokens = draft_tokens, a.tree_parent = tree_parent, a.tree_mask = tree_mask;
    a.node_count = node_count, a.match_len = match_len, a.status = status;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    a.part_hdr = reinterpret_cast<int2*>(ws + s.off_hdr);
    a.list_a = reinterpret_cast<uint32_t*>(ws + s.off_a);
    a.list_b = reinterpret_cast<uint32_t*>(ws + s.off_b);
    a.pool_tokens = p->pool_tokens;
    a.n_groups = p->n_groups, a.n_seq = p->n_seq, a.max_group_tokens = p->max_group_tokens;
    a.gamma_max = p->gamma_max, a.top_k = p->top_k, a.p_min = p->pattern_lookup_min, a.p_max = p->pattern_lookup_max;
    a.vocab = p->vocab, a.parts = s.parts, a.chunk = s.chunk, a.cap = s.cap, a.min_confidence = p->min_confidence;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipLaunchKernelGGL(seer::draft::draft_match_kernel, dim3(s.parts, p->n_groups), dim3(seer::draft::kMatchThreads), 0, stream, a,
                       p->B);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return static_cast<int>(err);
    hipLaunchKernelGGL(seer::draft::draft_expand_kernel, dim3(p->B), dim3(seer::draft::kThreads), 0, stream, a);
    err = hipGetLastError();
    return err == hipSuccess ? SEER_OK : static_cast<int>(err);
}

// ------------------------------------------------------------------------------------------------
// Appending the tokens a step emitted to the histories (the counterpart of the draft server's
// update call, Appendix A.2: new tokens of one request go to that request's own sequence).
// ------------------------------------------------------------------------------------------------
namespace seer {
namespace draft {

struct AppendArgs {
    int32_t* tokens;
    const int32_t* seq_start;
    int32_t* seq_len;
    const int32_t* seq_capacity;
    const int32_t* req_seq;
    const int32_t* emitted_tokens;
    const int32_t* n_emitted;
    int32_t* pattern;
    int32_t* pattern_len;
    int32_t* status;
    int64_t pool_tokens;
    int T, n_seq, p_max;
};

__global__ __launch_bounds__(64) void history_append_kernel(AppendArgs a) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int q = a.req_seq[b];
    int n = a.n_emitted[b];
    int bad = 0;
    int start = 0, len = 0;
    if (q < 0 || q >= a.n_seq) {
        bad = 1;
    } else {
        start = a.seq_start[q];
        len = a.seq_len[q];
        const int cap = a.seq_capacity[q];
        if (start < 0 || len < 0 || cap < len || static_cast<int64_t>(start) + cap > a.pool_tokens) bad = 1;
        else if (n < 0 || n > a.T || len + n > cap) bad = 2;
    }
    if (bad) {
        if (lane == 0 && a.status) atomicOr(a.status, bad);
        if (bad == 1) return;                        // no sequence to speak of: nothing is touched
        n = 0;                                       // no room (or a count out of range): nothing is appended
    }
    if (lane < n) a.tokens[start + len + lane] = a.emitted_tokens[static_cast<size_t>(b) * a.T + lane];
    const int total = len + n;
    if (lane == 0) {
        a.seq_len[q] = total;
        if (a.pattern_len) a.pattern_len[b] = min(total, a.p_max);
    }
    if (a.pattern && lane < a.p_max) {
        // the request's newest tokens, right-aligned: the appended ones come from the emitted row, the
        // older ones from the pool
        const int back = a.p_max - 1 - lane;         // 0 = the newest token
        int t = -1;
        if (back < n) t = a.emitted_tokens[static_cast<size_t>(b) * a.T + (n - 1 - back)];
        else if (back < total) t = a.tokens[start + total - 1 - back];
        a.pattern[static_cast<size_t>(b) * a.p_max + lane] = t;
    }
}

}  // namespace draft
}  // namespace seer

extern "C" int seer_history_append(int32_t* tokens, const int32_t* seq_start, int32_t* seq_len,
                                   const int32_t* seq_capacity, const int32_t* req_seq,
                                   const int32_t* emitted_tokens, const int32_t* n_emitted, int32_t B, int32_t T,
                                   int32_t n_seq, int64_t pool_tokens, int32_t pattern_lookup_max, int32_t* pattern,
                                   int32_t* pattern_len, int32_t* status, void* hip_stream) {
    if (B < 0 || n_seq < 1 || pool_tokens < 1) return SEER_EINVAL;
    if (T < 1 || T > SEER_MAX_T) return SEER_ESHAPE;
    if (pattern_lookup_max < 1 || pattern_lookup_max > seer::draft::kMaxPattern) return pattern_lookup_max < 1 ? SEER_EINVAL : SEER_EUNSUPPORTED;
    if (pool_tokens > 0x7fff0000ll) return SEER_EUNSUPPORTED;
    if (B == 0) return SEER_OK;
    if (!tokens || !seq_start || !seq_len || !seq_capacity || !req_seq || !emitted_tokens || !n_emitted) return SEER_EINVAL;
    if ((pattern == nullptr) != (pattern_len == nullptr)) return SEER_EINVAL;
    seer::draft::AppendArgs a{};
    a.tokens = tokens, a.seq_start = seq_start, a.seq_len = seq_len, a.seq_capacity = seq_capacity, a.req_seq = req_seq;
    a.emitted_tokens = emitted_tokens, a.n_emitted = n_emitted, a.pattern = pattern, a.pattern_len = pattern_len;
    a.status = status, a.pool_tokens = pool_tokens, a.T = T, a.n_seq = n_seq, a.p_max = pattern_lookup_max;
    hipLaunchKernelGGL(seer::draft::history_append_kernel, dim3(B), dim3(64), 0, static_cast<hipStream_t>(hip_stream), a);
    const hipError_t err = hipGetLastError();
    return err == hipSuccess ? SEER_OK : static_cast<int>(err);
}
