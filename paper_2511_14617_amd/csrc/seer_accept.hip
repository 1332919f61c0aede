// seer_accept: target token per verify slot (vocabulary argmax) and the longest
// accepted root path over the draft tree.
//
// The paper fixes what a verification step emits -- the accepted draft prefix
// plus one bonus token (Section 3.4.1; Table 2, whose acceptance lengths count
// the bonus token) -- and that with several candidate paths the longest
// accepted one counts (Section 3.4.2).  The scan below is the HBM-bound part:
// one pass over B*T*V fp32 logits.
//
// Kernel 1 (argmax_chunks): the rows are cut into chunks of 16 384 floats (8192 for small batches) so
//   that a launch has rows*chunks workgroups (thousands, against 256 CUs) no
//   matter how B*T and V split the work.  Each workgroup streams its chunk
//   with 16-byte loads, keeps (max, lowest index) per lane, reduces across the
//   wave with shuffles and across the 4 waves through LDS, and writes one
//   (value, index) pair.
// Kernel 2 (accept_walk): one workgroup per request.  The lanes of a slot share its chunk pairs, all
//   requested at once; then one wave walks the tree level by level: the accepted nodes of depth d + 1 are
//   the slots whose parent is an accepted node of depth d and whose draft token is that parent's target,
//   one ballot per level; the winner is the lowest slot of the last level that has any (a depth counts
//   deepest first, lowest slot on ties).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>
#include <utility>

#include "../../include/seer_verify.h"
#include "seer_device.h"
#include "seer_sampling.h"

namespace seer {

constexpr int kArgmaxThreads = 256;
// Floats per workgroup: 16 x 16-byte loads per lane, 8 where the launch would otherwise leave the chip without eight
// workgroups per CU.  Measured on V = 152 064, 16 384 against 8192 floats: greedy 52 vs 54 us for 576 rows, 364 vs 374 us
// for 4224 rows.  The sampled scan runs the generator for every load of a chunk, in the row or not, so its chunks are no longer
// than rows need: two loads for rows of up to 2048 (8192 rows of 1024 logits: 84 us with sixteen loads, 50 with eight, 28 with two).
// Its scalar form has no loads to keep in flight, only a loop, and is faster with more workgroups (1056 rows of 50 257 logits:
// 145 us with 16 384 floats each, 118 with 8192).
constexpr int kChunkLarge = 16384;
constexpr int kChunkSmall = 8192;
constexpr int kChunkShortRow = 2048;
constexpr int kFullLaunch = 2048;

__host__ __device__ inline int accept_num_chunks(int V, int chunk) { return (V + chunk - 1) / chunk; }
// the workspace holds the finer of the two partitions
__host__ __device__ inline int accept_max_chunks(int V) { return accept_num_chunks(V, kChunkSmall); }
inline int accept_chunk(int64_t rows, int V, bool sampled, bool vec4) {
    if (sampled && vec4 && V <= kChunkShortRow) return kChunkShortRow;
    if (sampled && (!vec4 || V <= kChunkSmall)) return kChunkSmall;
    return rows * accept_num_chunks(V, kChunkLarge) >= kFullLaunch ? kChunkLarge : kChunkSmall;
}

// (a, ia) beats (b, ib) iff a > b, or a == b and ia < ib.
__device__ __forceinline__ void take_better(float& v, int& i, float ov, int oi) {
    const bool better = (ov > v) || (ov == v && oi < i);
    v = better ? ov : v;
    i = better ? oi : i;
}

// f(0), f(1), .. with compile-time indices.
template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// Maximum over the lanes of a wave through DPP (rows of 16 lanes, then across them), in every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max_step(float v) {
    const int x = __float_as_int(v);
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(x, x, CTRL, ROW_MASK, 0xf, false)));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
    v = dpp_max_step<0x111, 0xf>(v);
    v = dpp_max_step<0x112, 0xf>(v);
    v = dpp_max_step<0x114, 0xf>(v);
    v = dpp_max_step<0x118, 0xf>(v);
    v = dpp_max_step<0x142, 0xa>(v);
    v = dpp_max_step<0x143, 0xc>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

// kSampled: the maximum is taken over logits[v] / tau + G(seed, row, v) (seer_sampling.h) instead of
// the logits themselves; one generator call serves the four elements of a 16-byte load.
struct SampleArgs {
    float inv_tau;
    uint32_t seed_lo, seed_hi;
};

// Upper bound of logits[v] / tau + G_v without the two logarithms: with z = the number of leading one bits of the
// generator's word (of its upper 23 bits, which are all that G uses), 1 - u > 2^-(z+1), so G < (z + 1) ln 2.
// kGumbelBoundC = ln 2 plus 0.05 for the error of the fixed-polynomial logarithms and for the roundings of the
// three fused multiply-adds involved (checked for every one of the 2^23 words on the host; the roundings stay
// below the slack while |logit / tau| < 2^17).  Beyond that range: a larger positive logit shows in the bound itself, which
// is then not relied on (kGumbelBoundMax); a larger negative one gives a value below -2^17 + 17, which cannot win
// as long as the value it is held against is above kGumbelSeenMin (else nothing is skipped).  A NaN never wins.
constexpr float kLn2 = 0.693147182f;
constexpr float kGumbelBoundC = 0.693147182f + 0.05f;
constexpr float kGumbelBoundMax = 130000.f;
constexpr float kGumbelSeenMin = -100000.f;
// (A bound per element: one bound for the four elements of a load, the largest logit with the most leading ones of the four
// words, costs half but lets enough more loads through to take 165 instead of 140 us on 1056 rows.)
__device__ __forceinline__ float perturb_upper_bound(float logit, float inv_tau, uint32_t w) {
    const int z = __builtin_clz(~w | 0x1ffu);          // 0 .. 23
    return __builtin_fmaf(static_cast<float>(z), kLn2, __builtin_fmaf(logit, inv_tau, kGumbelBoundC));
}

template <bool kVec4, bool kSampled, int kChunk>
__global__ __launch_bounds__(kArgmaxThreads) void argmax_chunks(const float* __restrict__ logits, int V,
                                                                int n_chunks, float* __restrict__ part_val,
                                                                int* __restrict__ part_idx, SampleArgs sa) {
    const int row = blockIdx.x / n_chunks;
    const int chunk = blockIdx.x - row * n_chunks;
    const int begin = chunk * kChunk;
    const int end = min(V, begin + kChunk);
    const float* __restrict__ base = logits + static_cast<size_t>(row) * V;

    float best = kNegInf;
    int best_i = begin;  // a row of -inf (or an all -inf chunk) resolves to its first index
    if constexpr (kVec4 && kSampled) {
        // The sampled scan is bound by its arithmetic, and what no element can do without is the generator and the
        // bound; the two polynomial logarithms are for elements that can win.  So a wave first takes the bound of
        // every one of its loads, then computes the exact values of the load that holds the largest bound, and the
        // best exact value of the workgroup's waves is what the other bounds are held against: an element whose upper bound
        // lies strictly below a perturbed value that has been computed is neither the maximum nor tied with it.
        // A handful of the workgroup's 64 loads reach the second computation (the generator is run again for them).
        // The result is that of the plain scan, bit for bit: only provable losers are skipped.
        // Measured, 1056 rows of 152 064 logits: 117 us; 158 us when every load was decided as it came (a third of them went
        // to the logarithms, the first of each wave always).
        constexpr int kIter = kChunk / (kArgmaxThreads * 4);
        constexpr int kWaves = kArgmaxThreads / kWave;
        __shared__ float s_seen[kWaves];                 // per wave: a perturbed value it has computed
        const int wv = threadIdx.x / kWave;
        using Loads = std::make_integer_sequence<int, kIter>;
        f32x4 x[kIter];
        for_each_index([&](auto ic) __attribute__((always_inline)) {
            constexpr int it = decltype(ic)::value;
            const int i = begin + (it * kArgmaxThreads + threadIdx.x) * 4;
            x[it] = (i < end) ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(base + i))
                              : f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
        }, Loads{});
        float ub[kIter], top = kNegInf;
        int top_it = 0;
        for_each_index([&](auto ic) __attribute__((always_inline)) {
            constexpr int it = decltype(ic)::value;
            const int i = begin + (it * kArgmaxThreads + threadIdx.x) * 4;
            const Philox4 r = philox4x32_10(static_cast<uint32_t>(i) >> 2, static_cast<uint32_t>(row), 0u, 0u, sa.seed_lo, sa.seed_hi);
            const float u0 = perturb_upper_bound(x[it].x, sa.inv_tau, r.w[0]);
            const float u1 = perturb_upper_bound(x[it].y, sa.inv_tau, r.w[1]);
            const float u2 = perturb_upper_bound(x[it].z, sa.inv_tau, r.w[2]);
            const float u3 = perturb_upper_bound(x[it].w, sa.inv_tau, r.w[3]);
            const float u4 = fmaxf(fmaxf(u0, u1), fmaxf(u2, u3));
            const float u = u4 < kGumbelBoundMax ? u4 : -kNegInf;          // (too large for the slack, or infinite: always computed)
            ub[it] = i < end ? u : kNegInf;
            if (ub[it] > top) top = ub[it], top_it = it;
            __builtin_amdgcn_sched_barrier(0);           // (load by load: interleaved, they take 6 % longer)
        }, Loads{});
        // the exact values of load `it` (uniform), every lane
        auto compute = [&](int it) __attribute__((always_inline)) {
            // (by masks: a chain of selects becomes one indexed load, and with it the array moves to scratch memory)
            u32x4 bits = {0u, 0u, 0u, 0u};
            for_each_index([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                bits |= __builtin_bit_cast(u32x4, x[k]) & (it == k ? 0xffffffffu : 0u);
            }, Loads{});
            const f32x4 y = __builtin_bit_cast(f32x4, bits);
            const int i = begin + (it * kArgmaxThreads + threadIdx.x) * 4;
            if (i >= end) return;
            const Philox4 r = philox4x32_10(static_cast<uint32_t>(i) >> 2, static_cast<uint32_t>(row), 0u, 0u, sa.seed_lo, sa.seed_hi);
#pragma unroll
            for (int c = 0; c < 4; ++c) take_better(best, best_i, perturb(y[c], sa.inv_tau, r.w[c]), i + c);
        };
        const uint64_t holders = __ballot(top == wave_max_dpp(top));
        int first = holders ? __builtin_amdgcn_readlane(top_it, __builtin_ctzll(holders)) : 0;
        uint32_t todo = 1u << first;
        bool exchanged = false;
        while (todo) {                                   // first the load with the largest bound, then what can still win
            const int it = __builtin_ctz(todo);
            todo &= todo - 1;
            compute(it);
            if (!exchanged) {
                exchanged = true;
                const float m = wave_max_dpp(best);
                if ((threadIdx.x & (kWave - 1)) == 0) s_seen[wv] = m;
                __syncthreads();                         // (once per wave, every wave)
                float seen = s_seen[0];
#pragma unroll
                for (int w = 1; w < kWaves; ++w) seen = fmaxf(seen, s_seen[w]);
                if (!(seen > kGumbelSeenMin)) seen = kNegInf;
                for_each_index([&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    if (k != first && __any(!(ub[k] < seen) && begin + (k * kArgmaxThreads + static_cast<int>(threadIdx.x)) * 4 < end))
                        todo |= 1u << k;
                }, Loads{});
            }
        }
    } else if constexpr (kVec4) {
        // V % 4 == 0 and a 16-byte aligned base: every row starts aligned.
        constexpr int kIter = kChunk / (kArgmaxThreads * 4);
        f32x4 x[kIter];
#pragma unroll
        for (int it = 0; it < kIter; ++it) {
            const int i = begin + (it * kArgmaxThreads + threadIdx.x) * 4;
            x[it] = (i < end) ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(base + i))
                              : f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
        }
#pragma unroll
        for (int it = 0; it < kIter; ++it) {
            const int i = begin + (it * kArgmaxThreads + threadIdx.x) * 4;
            if (i < end) {  // indices ascend within a lane: strict '>' keeps the lowest
                if (x[it].x > best) { best = x[it].x; best_i = i; }
                if (x[it].y > best) { best = x[it].y; best_i = i + 1; }
                if (x[it].z > best) { best = x[it].z; best_i = i + 2; }
                if (x[it].w > best) { best = x[it].w; best_i = i + 3; }
            }
        }
    } else {
        for (int i = begin + threadIdx.x; i < end; i += kArgmaxThreads) {
            float x = base[i];
            if constexpr (kSampled) {
                const Philox4 r = philox4x32_10(static_cast<uint32_t>(i) >> 2, static_cast<uint32_t>(row), 0u, 0u,
                                                sa.seed_lo, sa.seed_hi);
                x = perturb(x, sa.inv_tau, r.w[i & 3]);
            }
            if (x > best) { best = x; best_i = i; }
        }
    }
    // A lane that met nothing above -inf still reports (-inf, begin); that pair can only
    // win when the whole chunk is -inf, and then `begin` is the right answer.

#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(best_i, o, kWave);
        take_better(best, best_i, ov, oi);
    }
    __shared__ float s_val[kArgmaxThreads / kWave];
    __shared__ int s_idx[kArgmaxThreads / kWave];
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_val[wave] = best;
        s_idx[wave] = best_i;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kArgmaxThreads / kWave; ++w) take_better(best, best_i, s_val[w], s_idx[w]);
        part_val[blockIdx.x] = best;
        part_idx[blockIdx.x] = best_i;
    }
}

constexpr int kWalkThreads = 256;

__global__ __launch_bounds__(kWalkThreads) void accept_walk(const float* __restrict__ part_val,
                                                     const int* __restrict__ part_idx, int n_chunks,
                                                     const int32_t* __restrict__ draft_tokens,
                                                     const int32_t* __restrict__ tree_parent, int T, int log2_per_slot,
                                                     int32_t* __restrict__ accepted_len,
                                                     int32_t* __restrict__ accepted_path,
                                                     int32_t* __restrict__ bonus_token,
                                                     int32_t* __restrict__ target_argmax) {
    // Two short chains, launch aside: one round trip for the chunk pairs (2^log2_per_slot lanes per slot, up to eight
    // pairs each at a time), a few ballots for the tree.  With one lane per slot and a serial walk it took 4.8 us for 64
    // requests of 9 slots (10 chunks) and 7.4 us for 32 trees of 33 slots (19 chunks).
    __shared__ int s_tgt[SEER_MAX_T];
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const size_t row0 = static_cast<size_t>(b) * T;
    int draft = 0, par = -2;
    if (tid < T) {
        draft = draft_tokens[row0 + tid];
        par = tree_parent ? tree_parent[row0 + tid] : tid - 1;
    }
    const int slot = tid >> log2_per_slot, sub = tid & ((1 << log2_per_slot) - 1);
    float best = kNegInf;
    int best_i = 0x7fffffff;
    if (slot < T) {
        const size_t at = (row0 + slot) * n_chunks;
        for (int c = sub; c < n_chunks; c += 8 << log2_per_slot) {
            float v[8];
            int ix[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {               // (the ones past the end re-read the last pair)
                const int ck = min(c + (k << log2_per_slot), n_chunks - 1);
                v[k] = part_val[at + ck];
                ix[k] = part_idx[at + ck];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) take_better(best, best_i, v[k], ix[k]);
        }
    }
    for (int o = 1; o < (1 << log2_per_slot); o <<= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(best_i, o, kWave);
        take_better(best, best_i, ov, oi);
    }
    if (slot < T && sub == 0) {
        target_argmax[row0 + slot] = best_i;
        s_tgt[slot] = best_i;
    }
    __syncthreads();
    if (tid >= kWave) return;
    // lane t = slot t; a parent outside 0 .. t-1 counts as a padded slot (never accepted)
    const bool has_parent = tid > 0 && tid < T && par >= 0 && par < tid;
    if (!has_parent) par = 0;
    const bool match = has_parent && draft == s_tgt[par];
    uint64_t level = 1;                                  // accepted nodes of the current depth
    int len = 0, win = 0;
    for (;;) {
        const uint64_t next = __ballot(match && ((level >> par) & 1));
        if (!next) break;
        level = next;
        win = __builtin_ctzll(next);
        ++len;
    }
    int path = -1, node = win;
    for (int i = len; i >= 0; --i) {
        if (tid == i) path = node;
        node = __builtin_amdgcn_readlane(par, node);
    }
    if (tid < T) accepted_path[row0 + tid] = path;
    if (tid == 0) {
        accepted_len[b] = len;
        if (bonus_token) bonus_token[b] = s_tgt[win];
    }
}

}  // namespace seer

extern "C" size_t seer_accept_workspace(int32_t B, int32_t T, int32_t V) {
    if (B < 1 || T < 1 || T > SEER_MAX_T || V < 1) return 0;
    const size_t pairs = static_cast<size_t>(B) * T * seer::accept_max_chunks(V);
    return pairs * (sizeof(float) + sizeof(int32_t));
}

namespace seer {

// Argument checks that need no device: what both entry-point families share.
static int check_accept_args(const float* logits, const int32_t* draft_tokens, int32_t B, int32_t T, int32_t V,
                             const int32_t* accepted_len, const int32_t* accepted_path, const int32_t* target_token) {
    if (B < 0 || V < 1) return SEER_EINVAL;
    if (T < 1 || T > SEER_MAX_T) return SEER_ESHAPE;
    if (B == 0) return SEER_OK;
    if (!logits || !draft_tokens || !accepted_len || !accepted_path || !target_token) return SEER_EINVAL;
    if (static_cast<int64_t>(B) * T * accept_max_chunks(V) > 0x7fffffffLL) return SEER_ESHAPE;
    if (reinterpret_cast<uintptr_t>(logits) % 4 != 0) return SEER_EALIGN;
    return SEER_OK;
}

// The two launches.  scratch holds `capacity` (value, index) pairs: capacity floats, then capacity ints;
// the caller has checked that B * T * n_chunks pairs fit.
static int launch_accept(const float* logits, const int32_t* draft_tokens, const int32_t* tree_parent, int32_t B,
                         int32_t T, int32_t V, bool sampled, SampleArgs sa, int32_t* accepted_len,
                         int32_t* accepted_path, int32_t* bonus_token, int32_t* target_token, void* scratch,
                         size_t capacity, hipStream_t stream) {
    const bool vec4 = (V % 4 == 0) && (reinterpret_cast<uintptr_t>(logits) % 16 == 0);
    const int chunk = accept_chunk(static_cast<int64_t>(B) * T, V, sampled, vec4);
    const int n_chunks = accept_num_chunks(V, chunk);
    float* part_val = static_cast<float*>(scratch);
    int* part_idx = reinterpret_cast<int*>(part_val + capacity);
    const dim3 grid(static_cast<unsigned>(static_cast<size_t>(B) * T * n_chunks));
    const dim3 block(kArgmaxThreads);
#define SEER_SCAN(VEC4, SAMPLED, CHUNK)                                                                                       \
    if (vec4 == VEC4 && sampled == SAMPLED && chunk == CHUNK)                                                                 \
        hipLaunchKernelGGL((argmax_chunks<VEC4, SAMPLED, CHUNK>), grid, block, 0, stream, logits, V, n_chunks, part_val, part_idx, sa);
    SEER_SCAN(true, true, kChunkLarge)
    SEER_SCAN(true, true, kChunkSmall)
    SEER_SCAN(true, true, kChunkShortRow)
    SEER_SCAN(true, false, kChunkLarge)
    SEER_SCAN(true, false, kChunkSmall)
    SEER_SCAN(false, true, kChunkSmall)
    SEER_SCAN(false, false, kChunkLarge)
    SEER_SCAN(false, false, kChunkSmall)
#undef SEER_SCAN
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return static_cast<int>(err);
    int log2_per_slot = 0;                              // lanes per slot: a power of two that fits the workgroup and a wave
    while (log2_per_slot < 6 && (T << (log2_per_slot + 1)) <= kWalkThreads && (1 << log2_per_slot) < n_chunks) ++log2_per_slot;
    // no more waves than the lanes need (4096 requests of two slots, one chunk each: scan and walk 23.3 us with four waves, 22.0 with one)
    const int threads = ((T << log2_per_slot) + kWave - 1) / kWave * kWave;
    hipLaunchKernelGGL(accept_walk, dim3(B), dim3(threads), 0, stream, part_val, part_idx, n_chunks, draft_tokens,
                       tree_parent, T, log2_per_slot, accepted_len, accepted_path, bonus_token, target_token);
    err = hipGetLastError();
    return err == hipSuccess ? SEER_OK : static_cast<int>(err);
}

static int run_accept(const float* logits, const int32_t* draft_tokens, const int32_t* tree_parent, int32_t B,
                      int32_t T, int32_t V, bool sampled, SampleArgs sa, int32_t* accepted_len,
                      int32_t* accepted_path, int32_t* bonus_token, int32_t* target_token, void* workspace,
                      size_t workspace_bytes, void* hip_stream) {
    const int rc = check_accept_args(logits, draft_tokens, B, T, V, accepted_len, accepted_path, target_token);
    if (rc != SEER_OK || B == 0) return rc;
    const size_t need = seer_accept_workspace(B, T, V);
    if (!workspace || workspace_bytes < need) return SEER_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return SEER_EALIGN;
    const size_t capacity = static_cast<size_t>(B) * T * accept_max_chunks(V);     // pairs the workspace holds
    return launch_accept(logits, draft_tokens, tree_parent, B, T, V, sampled, sa, accepted_len, accepted_path,
                         bonus_token, target_token, workspace, capacity, static_cast<hipStream_t>(hip_stream));
}

}  // namespace seer

extern "C" int seer_accept(const float* logits, const int32_t* draft_tokens, const int32_t* tree_parent,
                           int32_t B, int32_t T, int32_t V, int32_t* accepted_len, int32_t* accepted_path,
                           int32_t* bonus_token, int32_t* target_argmax, void* workspace,
                           size_t workspace_bytes, void* hip_stream) {
    return seer::run_accept(logits, draft_tokens, tree_parent, B, T, V, false, seer::SampleArgs{1.f, 0u, 0u},
                            accepted_len, accepted_path, bonus_token, target_argmax, workspace, workspace_bytes,
                            hip_stream);
}

extern "C" int seer_accept_sampled(const float* logits, const int32_t* draft_tokens, const int32_t* tree_parent,
                                   int32_t B, int32_t T, int32_t V, float temperature, uint64_t seed,
                                   int32_t* accepted_len, int32_t* accepted_path, int32_t* bonus_token,
                                   int32_t* target_token, void* workspace, size_t workspace_bytes,
                                   void* hip_stream) {
    if (!(temperature > 0.f) || temperature > 3.0e38f) return SEER_EINVAL;   // positive and finite
    const seer::SampleArgs sa{1.0f / temperature, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
    return seer::run_accept(logits, draft_tokens, tree_parent, B, T, V, true, sa, accepted_len, accepted_path,
                            bonus_token, target_token, workspace, workspace_bytes, hip_stream);
}

// ---------------------------------------------------------------------------
// seer_accept_static: seer_accept for callers that cannot allocate.  The chunk results of the scan live in
// a fixed array in the library's own device image instead of a caller workspace.
// ---------------------------------------------------------------------------
namespace seer {

constexpr size_t kStaticPairs = size_t{SEER_ACCEPT_STATIC_MAX_PAIRS};      // (value, index) pairs
static __device__ __align__(256) unsigned char scratch[kStaticPairs * (sizeof(float) + sizeof(int32_t))];

// In host code `scratch` is only a stand-in for the symbol, not a device address; every GPU holds its own
// copy of the array at its own address, looked up once per device and kept here.
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static void* g_scratch_ptr[kMaxDevices];

static int static_scratch(void** ptr) {
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return static_cast<int>(err);
    if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return static_cast<int>(err);
        if (!p) return static_cast<int>(hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return SEER_OK;
}

}  // namespace seer

extern "C" int seer_accept_static(const float* logits, const int32_t* draft_tokens, const int32_t* tree_parent,
                                  int32_t B, int32_t T, int32_t V, int32_t* accepted_len, int32_t* accepted_path,
                                  int32_t* bonus_token, int32_t* target_argmax, void* hip_stream) {
    const int rc = seer::check_accept_args(logits, draft_tokens, B, T, V, accepted_len, accepted_path, target_argmax);
    if (rc != SEER_OK) return rc;
    const size_t pairs = static_cast<size_t>(B) * T * seer::accept_num_chunks(V, seer::kChunkLarge);
    if (pairs > seer::kStaticPairs) return SEER_ELIMIT;
    void* ptr = nullptr;
    const int rs = seer::static_scratch(&ptr);      // also with B == 0: resolves the address, launches nothing
    if (rs != SEER_OK || B == 0) return rs;
    // Every pair the walk reads is written by this call's scan first, so nothing has to start at zero.
    return seer::launch_accept(logits, draft_tokens, tree_parent, B, T, V, false, seer::SampleArgs{1.f, 0u, 0u},
                               accepted_len, accepted_path, bonus_token, target_argmax, ptr, seer::kStaticPairs,
                               static_cast<hipStream_t>(hip_stream));
}
