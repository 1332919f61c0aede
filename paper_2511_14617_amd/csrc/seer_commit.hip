// seer_kv_commit: the step right after verification.
//
// A verify step scores T = gamma + 1 positions whose keys/values sit at the request's last T
// logical positions, slot s at n0 + s.  With several candidate paths (Section 3.4.2, multi-path
// drafting) one root path is accepted; the sequence must continue exactly as serial decoding
// would have produced it (Section 3.1, lossless), i.e. prefix + root + accepted draft tokens in
// path order.  So the rows of path[1..a] move to positions n0+1 .. n0+a, the length becomes
// n0 + 1 + a, and the step emits the a accepted draft tokens plus the bonus token (Section
// 3.4.1).  For a linear chain path[i] = i and nothing moves.
//
// One workgroup per request.  It reads the rows to move into registers, for as many KV heads at once as its threads
// hold, waits for the whole workgroup, then writes them (a destination may be another row's source, of the same head).  The
// amount of data is tiny (at most 63 rows of 256..1152 bytes per head), so what bounds it is the chain of
// dependent loads: lengths and path, block table, rows.  Rows already in place are not read.  (With 256 threads, one head after the
// other and the block table looked up for every chunk it took 10.2 us for 16 chains on eight heads, where nothing moves.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/seer_verify.h"
#include "seer_device.h"

namespace seer {

constexpr int kCommitThreads = 1024;
constexpr int kCommitHold = 5;            // 16-byte chunks a thread holds
constexpr int kCommitMaxChunks = 4608;    // 16-byte chunks of one head's rows, at most: 63 rows x 72, with some room
static_assert(kCommitMaxChunks <= kCommitThreads * kCommitHold, "the rows of one head fit");

struct CommitArgs {
    unsigned char* k_pages;
    unsigned char* v_pages;          // nullptr: shared latent
    const int32_t* block_table;
    int32_t* ctx_len;
    const int32_t* accepted_len;
    const int32_t* accepted_path;
    const int32_t* draft_tokens;     // may be nullptr (then nothing is emitted)
    const int32_t* bonus_token;
    int32_t* emitted_tokens;
    int32_t* n_emitted;
    int32_t* status;                 // may be nullptr
    int T, Hkv, P, num_pages, max_pages;
    int k_chunks, v_chunks;          // 16-byte chunks per K row, per V row
};

__global__ __launch_bounds__(kCommitThreads) void kv_commit_kernel(CommitArgs a) {
    __shared__ int s_path[SEER_MAX_T];
    __shared__ int2 s_page[SEER_MAX_T], s_slot[SEER_MAX_T];   // path node i: page and slot of its source and of its destination
    __shared__ int s_draft[SEER_MAX_T];
    __shared__ int s_flags;           // status bits, kMoves
    constexpr int kMoves = 8;
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int T = a.T;
    const int n = a.ctx_len[b];
    const int n0 = n - T;
    const int len = a.accepted_len[b];
    // (the tokens to emit are requested beside the lengths and the path, not behind them)
    const int bonus = a.emitted_tokens ? a.bonus_token[b] : 0;
    if (tid == 0) s_flags = 0;
    if (tid < T) {
        s_path[tid] = a.accepted_path[static_cast<size_t>(b) * T + tid];
        if (a.emitted_tokens) s_draft[tid] = a.draft_tokens[static_cast<size_t>(b) * T + tid];
    }
    __syncthreads();
    // a request whose inputs are out of range is left as it is and reported
    int bad = 0;
    if (n < T || (static_cast<int64_t>(n) + a.P - 1) / a.P > a.max_pages) bad |= 1;
    if (len < 0 || len > T - 1) bad |= 4;
    if (!bad && tid <= len) {
        const int node = s_path[tid];
        // a node is used as an index only once it is known to lie on an ascending path inside the T slots
        const bool node_ok = tid == 0 ? node == 0 : (node > s_path[tid - 1] && node > 0 && node < T);
        if (!node_ok) atomicOr(&s_flags, 4);
        if (tid >= 1 && node_ok) {
            const int32_t* table = a.block_table + static_cast<size_t>(b) * a.max_pages;
            const int l_src = (n0 + node) / a.P, l_dst = (n0 + tid) / a.P;
            const int p_src = table[l_src], p_dst = table[l_dst];
            if (node != tid) atomicOr(&s_flags, kMoves);
            if (p_src < 0 || p_src >= a.num_pages || p_dst < 0 || p_dst >= a.num_pages) atomicOr(&s_flags, 2);
            s_page[tid] = make_int2(p_src, p_dst);
            s_slot[tid] = make_int2(n0 + node - l_src * a.P, n0 + tid - l_dst * a.P);
        }
    }
    __syncthreads();
    const int flags = s_flags;       // (one read: a second word cost trees 0.1 us)
    bad |= flags & ~kMoves;
    if (bad) {                       // uniform for the workgroup
        if (tid == 0 && a.status) atomicOr(a.status, bad);
        return;
    }

    // Where every accepted row is in place already (a chain) nothing is left but the lengths and the tokens: the divisions of
    // sixteen waves find nothing to move (16 requests of 9 slots, with the tokens requested early: 5.3 -> 4.8 us on the device).
    const int per_tok = a.k_chunks + a.v_chunks;
    const int per_head = len * per_tok;
    const int heads_at_once = per_head ? min(a.Hkv, kCommitThreads * kCommitHold / per_head) : a.Hkv;
    for (int h0 = 0; h0 < a.Hkv && (flags & kMoves); h0 += heads_at_once) {
        const int total = min(heads_at_once, a.Hkv - h0) * per_head;
        u32x4 hold[kCommitHold];
        unsigned char* dst[kCommitHold];
#pragma unroll
        for (int j = 0; j < kCommitHold; ++j) {
            const int idx = tid + j * kCommitThreads;
            dst[j] = nullptr;
            if (idx < total) {
                const int h = idx / per_head, in_head = idx - h * per_head;
                const int i = 1 + in_head / per_tok, c = in_head - (i - 1) * per_tok;
                if (s_path[i] != i) {                  // already in place otherwise
                    const int2 page = s_page[i], slot = s_slot[i];
                    const size_t src_row = (static_cast<size_t>(page.x) * a.Hkv + h0 + h) * a.P + slot.x;
                    const size_t dst_row = (static_cast<size_t>(page.y) * a.Hkv + h0 + h) * a.P + slot.y;
                    const bool is_k = c < a.k_chunks;
                    unsigned char* base = is_k ? a.k_pages : a.v_pages;
                    const size_t chunks = is_k ? a.k_chunks : a.v_chunks, at = is_k ? c : c - a.k_chunks;
                    hold[j] = *reinterpret_cast<const u32x4*>(base + (src_row * chunks + at) * 16);
                    dst[j] = base + (dst_row * chunks + at) * 16;
                }
            }
        }
        __syncthreads();             // every source row of these heads has been read
#pragma unroll
        for (int j = 0; j < kCommitHold; ++j)
            if (dst[j]) *reinterpret_cast<u32x4*>(dst[j]) = hold[j];
    }
    if (tid == 0) a.ctx_len[b] = n0 + 1 + len;
    if (a.emitted_tokens && tid < T) {
        int tok = -1;
        if (tid < len) tok = s_draft[s_path[tid + 1]];
        else if (tid == len) tok = bonus;
        a.emitted_tokens[static_cast<size_t>(b) * T + tid] = tok;
        if (tid == 0) a.n_emitted[b] = len + 1;
    }
}

}  // namespace seer

extern "C" int seer_kv_commit(const seer_attn_params* p, void* k_pages, void* v_pages, const int32_t* block_table,
                              int32_t* ctx_len, const int32_t* accepted_len, const int32_t* accepted_path,
                              const int32_t* draft_tokens, const int32_t* bonus_token, int32_t* emitted_tokens,
                              int32_t* n_emitted, int32_t* status, void* hip_stream) {
    if (!p) return SEER_EINVAL;
    if (p->B < 0 || p->num_pages < 1 || p->max_pages_per_seq < 1 || p->page_size < 1) return SEER_EINVAL;
    if (p->T < 1 || p->T > SEER_MAX_T || p->Hkv < 1 || p->Dqk < 1) return SEER_ESHAPE;
    const bool shared = p->kv_shared_latent != 0;
    if (!shared && p->Dv < 1) return SEER_ESHAPE;
    if (p->Dqk % 8 != 0 || (!shared && p->Dv % 8 != 0)) return SEER_ESHAPE;            // rows are moved in 16-byte chunks
    if (p->B == 0) return SEER_OK;
    if (!k_pages || (!shared && !v_pages) || !block_table || !ctx_len || !accepted_len || !accepted_path) return SEER_EINVAL;
    if (emitted_tokens && (!draft_tokens || !bonus_token || !n_emitted)) return SEER_EINVAL;
    if (reinterpret_cast<uintptr_t>(k_pages) % 16 != 0 || (!shared && reinterpret_cast<uintptr_t>(v_pages) % 16 != 0))
        return SEER_EALIGN;
    seer::CommitArgs a{};
    a.k_pages = static_cast<unsigned char*>(k_pages);
    a.v_pages = shared ? nullptr : static_cast<unsigned char*>(v_pages);
    a.block_table = block_table;
    a.ctx_len = ctx_len;
    a.accepted_len = accepted_len;
    a.accepted_path = accepted_path;
    a.draft_tokens = draft_tokens;
    a.bonus_token = bonus_token;
    a.emitted_tokens = emitted_tokens;
    a.n_emitted = n_emitted;
    a.status = status;
    a.T = p->T, a.Hkv = p->Hkv, a.P = p->page_size, a.num_pages = p->num_pages, a.max_pages = p->max_pages_per_seq;
    a.k_chunks = p->Dqk / 8;
    a.v_chunks = shared ? 0 : p->Dv / 8;
    if (static_cast<int64_t>(p->T - 1) * (a.k_chunks + a.v_chunks) > seer::kCommitMaxChunks) return SEER_EUNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipLaunchKernelGGL(seer::kv_commit_kernel, dim3(p->B), dim3(seer::kCommitThreads), 0, stream, a);
    const hipError_t err = hipGetLastError();
    return err == hipSuccess ? SEER_OK : static_cast<int>(err);
}
