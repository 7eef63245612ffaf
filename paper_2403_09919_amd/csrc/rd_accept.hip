// rd_accept: greedy verification (Sec. 3.4, Fig. 2) for gfx950 in one launch.
//
// Phase 1 (all workgroups): the valid logit rows (p < n_packed[b]) are cut into chunks of
// a few thousand floats; a workgroup streams one chunk with 16-byte loads, reduces it to
// (max value, smallest index attaining it), the row's 64-bit key in the workspace: stored where the row is
// one chunk, folded in with one device-scope atomic max, and waited for, where it is several.  The key orders
// (value, -index), so the row's final key is its arg max with the smallest-index tie rule.  This phase is a pure
// HBM stream over the valid logits.
// Phase 2 (the workgroup that completes a sequence, found with a per-row and then a
// per-sequence counter): decodes the row keys, writes the arg maxes, compares every candidate token with the
// prediction at its parent (a bit each), takes a candidate's accepted prefix as the run of ones from its first
// token, picks the best candidate with a wave-wide max on (length, -w) and writes the accepted slots and the next token.
// Up to 64 tokens one wave does all of phase 2 in registers: beside the round trips to memory it is bound by the
// number of its instructions (1.7 ns each in a lone wave).  us per launch, phase 2 through LDS, barriers that waited for
// stores and a walk over every candidate's tokens -> now: 4 x 4 tokens, V = 1000 4.65 -> 3.60; 8 x 5, 32000
// 6.5 -> 5.9; 70 x 5 12.9 -> 11.4; 16 sequences of 16 x 5 22.0 -> 21.3.
// Two counter levels keep the number of atomics that hit one address small (chunks per row,
// rows per sequence); hundreds of increments of a single word would serialise and cost more
// than the stream itself.
#include "rd_internal.h"
#include <cstdlib>

RD_TRACE_DEFINE(rd_debug_set_trace_accept)

namespace {

constexpr int kAccThreads = 256;
constexpr int kMaxChunks = 64;

struct AccPlan {
    int chunks;       // chunks per logit row
    int chunk_len;    // floats per chunk (multiple of 1024)
    int loads;        // 16-byte loads per thread issued together (1, 2, 4, ..., 32)
    int speculate;    // 1: first loads before the packed count is known (small logit tensors)
    size_t row_counters_off, keys_off;   // byte offsets in the workspace (sequence counters at 0)
    size_t total_bytes;                  // all of it must be zero between calls (and is left so)
};

// A workgroup issues all loads of its chunk at once: `loads` 16-byte loads per thread, so a chunk
// is 1024*loads floats.  Measured on MI355X (V = 32000): 4 or 8 loads per thread (8 or 4 chunks per
// row) are best from 22 to 500 valid rows -- 6.6 us and 21 us per launch against 10.6 us and 54 us
// with one load per thread, where the extra workgroups and the 32 atomics per row dominate, and
// 10 us and 27 us with one workgroup per row, where a workgroup's own streaming rate does.
AccPlan acc_plan(int B, int N, int V)
{
    AccPlan p;
    static const int loads_env = rd::env_int("RD_ACCEPT_LOADS", 0);      // tuning builds only
    int loads = ((long long)B * N >= 512) ? 8 : 4;
    if (loads_env == 1 || loads_env == 2 || loads_env == 4 || loads_env == 8 || loads_env == 16 || loads_env == 32) loads = loads_env;
    while ((V + 1024 * loads - 1) / (1024 * loads) > kMaxChunks) loads *= 2;     // huge vocabularies: the kernel loops
    p.loads = loads > 32 ? 32 : loads;
    static const int spec_env = rd::env_int("RD_ACCEPT_SPEC", -1);       // tuning builds only
    p.speculate = ((double)B * N * V * sizeof(float) <= 8e6 && p.loads <= 8) ? 1 : 0;
    if (spec_env >= 0) p.speculate = spec_env ? 1 : 0;
    int len = 1024 * loads;
    p.chunk_len = len;
    p.chunks = (V + len - 1) / len;
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    p.row_counters_off = up((size_t)B * sizeof(uint32_t));
    p.keys_off = p.row_counters_off + up((size_t)B * N * sizeof(uint32_t));
    p.total_bytes = p.keys_off + up((size_t)B * N * sizeof(unsigned long long));
    return p;
}

// (value, index) ordering of the arg max with the smallest-index tie rule.
__device__ __forceinline__ bool better(float v, int i, float bv, int bi)
{
    return v > bv || (v == bv && i < bi);
}

// Order-preserving 64-bit key of (value, index): larger value first, then smaller index.
// Every key of a real element is greater than 0, the cleared state of the workspace.
// (The index is -1 where the upper half is 0: no element compared.)
// -0.0 and +0.0 are one value to the comparison that defines the arg max, so both get +0.0's key.
__device__ __forceinline__ unsigned long long encode_key(float v, int i)
{
    const uint32_t u = (v == 0.0f) ? 0u : __float_as_uint(v);
    const uint32_t mono = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)mono << 32) | (uint32_t)~(uint32_t)i;
}
__device__ __forceinline__ int key_index(unsigned long long k) { return k >> 32 ? (int)~(uint32_t)k : -1; }

// Device-scope arrival: true for the thread whose increment brought the counter to `expected`.  What a thread has sent
// to other addresses could otherwise complete after its increment: a key that several chunks share (atomic max) and a
// lower-level counter have been waited for (wait_dev_stores; the returned value), or the workgroup that sees the full count
// would read a key that lacks a chunk.  A key that one workgroup alone stores need not be: it is never 0, the cleared state,
// and whoever sees the full count reads it until it is there (it was issued before the increment).
__device__ __forceinline__ bool arrive(uint32_t *counter, uint32_t expected)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    const uint32_t prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return prev + 1u == expected;
}

// SPEC: the first batch of logit loads is issued before n_packed[b] is known (every row of the [B,N,V] tensor is
// allocated, so a row beyond the packed count is read and dropped): one dependent round trip less in front
// of the stream.  For launches whose whole logit tensor is a few MB, where the extra rows cost nothing.
// With eight loads per thread the registers allow eight waves per SIMD and seven are faster where they end in the same
// round of workgroups (B=16, W=16, us: V=32000 23.5 -> 23.0, V=32768 24.1 -> 23.4; B=24, W=16, V=32000 29.3 -> 29.8).
template <int U, bool SPEC>
__global__ __launch_bounds__(kAccThreads) __attribute__((amdgpu_waves_per_eu(1, U == 8 ? 7 : 8))) void rd_accept_kernel(
    const float *__restrict__ logits, const int32_t *__restrict__ beams,
    const int32_t *__restrict__ unpack_index, const int32_t *__restrict__ n_packed,
    const int32_t *__restrict__ root_token, int W, int L, int V, int chunks, int chunk_len, uint32_t inv_l,
    int32_t *__restrict__ argmax_out, int32_t *__restrict__ n_accept, int32_t *__restrict__ best_beam,
    int32_t *__restrict__ best_len, int32_t *__restrict__ next_token, int32_t *__restrict__ accepted_idx,
    uint32_t *seq_counters, uint32_t *row_counters, unsigned long long *row_keys)
{
    __shared__ float s_val[kAccThreads / 64];
    __shared__ int s_idx[kAccThreads / 64];
    __shared__ int s_am[RD_MAX_N];
    __shared__ int s_slot[RD_MAX_N];
    __shared__ uint32_t s_seq_last;
    __shared__ unsigned long long s_ok[2 * kAccThreads / 64];
    __shared__ int s_best[2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = blockIdx.x, p = blockIdx.y, b = blockIdx.z;
    const int N = W * L;
    const float *row = logits + ((size_t)b * N + p) * V;
    const int v0 = chunk * chunk_len;
    const int v1 = min(V, v0 + chunk_len);
    float4 x0[U];
    int i0[U];
    if (SPEC && V >= 4) {
#pragma unroll
        for (int u = 0; u < U; ++u) x0[u] = rd::row4_at(row, v0 + (u * kAccThreads + tid) * 4, V, &i0[u]);
    }
    int P = n_packed[b];
    P = P < 1 ? 1 : (P > N ? N : P);
    if (p >= P) return;                                   // whole workgroup: row is padding
    RD_TR(0);

    // The candidates and their slots are only needed by the workgroup that ends up finishing the
    // sequence, but nobody knows which one that is: every workgroup fetches them now (a few
    // hundred bytes, overlapped with the logit stream) instead of paying two dependent round
    // trips to memory per accepted token at the very end.
    constexpr int kPre = (RD_MAX_N + kAccThreads - 1) / kAccThreads;     // tokens per thread
    int my_beam[kPre], my_slot[kPre], my_parent = 0, my_root = 0;        // (the parent is the token before)
    bool first[kPre];
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const int e = min(u * kAccThreads + tid, N - 1);
        my_beam[u] = beams[(size_t)b * N + e];
        my_slot[u] = unpack_index[(size_t)b * N + e];
        first[u] = (int)((uint32_t)e * inv_l >> 20) * L == e;
    }
    const bool one_wave = N <= 64;                        // uniform: the first wave finishes the sequence
    if (one_wave) my_parent = unpack_index[(size_t)b * N + min(max(tid - 1, 0), N - 1)];
    if (root_token != nullptr) my_root = root_token[b];

    // ---- phase 1: this chunk's (max, first index) -> the row's key ---------------------------------
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    if (V >= 4) {
        // U loads per thread in flight together; past the end of the row they are its last entries once more, whose keys
        // are those they had before
        for (int base = v0; base < v1; base += kAccThreads * 4 * U) {
            float4 x[U];
            int v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (SPEC && base == v0) { x[u] = x0[u]; v[u] = i0[u]; }
                else x[u] = rd::row4_at(row, base + (u * kAccThreads + tid) * 4, V, &v[u]);
            }
            // the largest value, then the first entry that holds it (v ascends with u)
            float m = -INFINITY;
#pragma unroll
            for (int u = 0; u < U; ++u) m = fmaxf(fmaxf(fmaxf(m, x[u].x), fmaxf(x[u].y, x[u].z)), x[u].w);
            int first_m = 0x7fffffff;
#pragma unroll
            for (int u = U - 1; u >= 0; --u) {
                int c = -1;
                c = x[u].w == m ? 3 : c;
                c = x[u].z == m ? 2 : c;
                c = x[u].y == m ? 1 : c;
                c = x[u].x == m ? 0 : c;
                first_m = c >= 0 ? v[u] + c : first_m;
            }
            if (better(m, first_m, bv, bi)) { bv = m; bi = first_m; }
        }
    } else {
        for (int v = v0 + tid; v < v1; v += kAccThreads) {
            const float x = row[v];
            if (better(x, v, bv, bi)) { bv = x; bi = v; }
        }
    }
    {   // the wave's largest value, then the smallest index that holds it
        const float m = rd::wave_reduce_max(bv);
        const uint32_t i = bv == m ? (uint32_t)bi : 0x7fffffffu;
        bi = (int)rd::wave_reduce_min_u(i);
        bv = m;
    }
    RD_TR(1);
    if (lane == 0) { s_val[wave] = bv; s_idx[wave] = bi; }
    rd_lds_barrier();
    if (one_wave && wave != 0) return;
    const size_t rowid = (size_t)b * N + p;
    uint32_t last = 0;
    if (tid == 0) {
        for (int w = 1; w < kAccThreads / 64; ++w)
            if (better(s_val[w], s_idx[w], bv, bi)) { bv = s_val[w]; bi = s_idx[w]; }
        // (a chunk without any value that compares, all NaN, leaves the lowest key)
        const unsigned long long key = bi != 0x7fffffff ? encode_key(bv, bi) : 1ull;
        if (chunks == 1) {                                             // the row is this workgroup's alone
            __hip_atomic_store(row_keys + rowid, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = arrive(seq_counters + b, (uint32_t)P) ? 1u : 0u;
        } else {
            __hip_atomic_fetch_max(row_keys + rowid, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            rd::wait_dev_stores();
            if (arrive(row_counters + rowid, (uint32_t)chunks)) {      // this row is complete
                row_counters[rowid] = 0;                               // ready for the next call
                last = arrive(seq_counters + b, (uint32_t)P) ? 1u : 0u;    // ... and so is the sequence
            }
        }
    }
    RD_TR(2);
    unsigned long long *seq_keys = row_keys + (size_t)b * N;
    auto row_argmax = [&](int r) __attribute__((always_inline)) {
        const unsigned long long key = rd::poll([&]() { return __hip_atomic_load(seq_keys + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                                                [](unsigned long long k) { return k != 0; });      // (its store is on its way: see arrive)
        return key_index(key);
    };
    static_assert(RD_MAX_W <= 128 && RD_MAX_N < (1 << 15), "candidates: two waves, index in 8 bits");

    // ---- phase 2 (last workgroup of the sequence): arg maxes, then token matching -----------------------
    if (one_wave) {
        // Lane = row, then token, then candidate; nothing goes through LDS.  A wave issues an instruction every 1.7 ns, so
        // that this part is as long as its code.
        if (!__builtin_amdgcn_readfirstlane(last)) return;
        RD_TR(3);
        const int am = lane < P ? row_argmax(lane) : -1;
        RD_TR(4);
        if (lane < N) argmax_out[(size_t)b * N + lane] = am;
        if (lane < P) seq_keys[lane] = 0;     // ready for the next call
        if (lane == 0) seq_counters[b] = 0;
        const int predicted = __builtin_amdgcn_ds_bpermute(min(max(my_parent, 0), N - 1) * 4, am);
        const bool ok = lane < N && (first[0] ? root_token == nullptr || my_beam[0] == my_root : predicted == my_beam[0]);
        const unsigned long long agree = __ballot(ok);
        // a candidate's accepted prefix is the run of ones from its first bit
        int len = 0;
        if (lane < W) {
            len = rd::accepted_run(agree, lane * L, L);
            n_accept[(size_t)b * W + lane] = len;
        }
        const int key = rd::wave_reduce_max_i(lane < W ? (len << 8) | (255 - lane) : 0);     // longest, smallest index among equals
        const int bl = key >> 8, bw = 255 - (key & 255);
        const int slot = __builtin_amdgcn_ds_bpermute((bw * L + min(lane, L - 1)) * 4, min(max(my_slot[0], 0), N - 1));
        if (lane < L) accepted_idx[(size_t)b * L + lane] = lane < bl ? slot : -1;
        const int next = __builtin_amdgcn_ds_bpermute(slot * 4, am);
        if (lane == max(bl - 1, 0)) {
            best_beam[b] = bw;
            best_len[b] = bl;
            next_token[b] = bl > 0 ? next : my_root;
        }
        RD_TR(5);
        return;
    }
    if (tid == 0) s_seq_last = last;
    rd_lds_barrier();
    if (!s_seq_last) return;
    RD_TR(3);
    for (int r = tid; r < N; r += kAccThreads) {
        const int am = r < P ? row_argmax(r) : -1;
        s_am[r] = am;
        argmax_out[(size_t)b * N + r] = am;
    }
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const int e = u * kAccThreads + tid;
        if (e < N) s_slot[e] = min(max(my_slot[u], 0), N - 1);
    }
    rd_lds_barrier();                                      // every key has been read
    RD_TR(4);
    for (int r = tid; r < P; r += kAccThreads) seq_keys[r] = 0;     // ready for the next call
    if (tid == 0) seq_counters[b] = 0;
    // one thread per candidate token: does the LLM agree with it; a bit each
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        const bool ok = u * kAccThreads + tid < N &&
                        (first[u] ? root_token == nullptr || my_beam[u] == my_root : s_am[s_slot[u * kAccThreads + tid - 1]] == my_beam[u]);
        const unsigned long long bits = __ballot(ok);
        if (lane == 0) s_ok[u * (kAccThreads / 64) + wave] = bits;
    }
    rd_lds_barrier();
    int len = 0;                                           // one thread per candidate
    if (tid < W) {
        len = rd::accepted_run(s_ok, tid * L, L);
        n_accept[(size_t)b * W + tid] = len;
    }
    if (wave < 2) {
        const int most = rd::wave_reduce_max_i(tid < W ? (len << 8) | (255 - tid) : 0);
        if (lane == 0) s_best[wave] = most;
    }
    rd_lds_barrier();
    const int key = max(s_best[0], s_best[1]);
    const int bl = key >> 8;
    const int bw = 255 - (key & 255);
    const int *bui = s_slot + bw * L;
    for (int t = tid; t < L; t += kAccThreads) accepted_idx[(size_t)b * L + t] = (t < bl) ? bui[t] : -1;
    if (tid == 0) {
        best_beam[b] = bw;
        best_len[b] = bl;
        next_token[b] = (bl > 0) ? s_am[bui[bl - 1]] : my_root;
    }
    RD_TR(5);
}

}  // namespace

extern "C" size_t rd_accept_workspace(int B, int W, int L, int V)
{
    if (rd_check_beam_shape(B, W, L) != RD_OK || V <= 0) return 0;
    return acc_plan(B, W * L, V).total_bytes;
}

// Argument checks shared by the two entry points; *plan is filled on success.
static int accept_check(const float *logits, const int32_t *beams, const int32_t *unpack_index,
                        const int32_t *n_packed, int B, int W, int L, int V,
                        const int32_t *argmax_out, const int32_t *n_accept, const int32_t *best_beam,
                        const int32_t *best_len, const int32_t *next_token, const int32_t *accepted_idx, AccPlan *plan)
{
    const int st = rd_check_beam_shape(B, W, L);
    if (st != RD_OK) return st;
    if (V <= 0) return RD_ERR_INVALID_ARG;
    if (B > 65535) return RD_ERR_UNSUPPORTED;
    if (!logits || !beams || !unpack_index || !n_packed || !argmax_out || !n_accept || !best_beam ||
        !best_len || !next_token || !accepted_idx)
        return RD_ERR_INVALID_ARG;
    if (!rd_aligned(logits, 16)) return RD_ERR_INVALID_ARG;
    *plan = acc_plan(B, W * L, V);
    return RD_OK;
}

// Enqueues the kernel on a zeroed workspace of plan.total_bytes at `ws`.
static int accept_launch(const AccPlan &plan, const float *logits, const int32_t *beams, const int32_t *unpack_index,
                         const int32_t *n_packed, const int32_t *root_token, int B, int W, int L, int V,
                         int32_t *argmax_out, int32_t *n_accept, int32_t *best_beam, int32_t *best_len,
                         int32_t *next_token, int32_t *accepted_idx, unsigned char *ws, hipStream_t stream)
{
    const int N = W * L;
    const dim3 grid(plan.chunks, N, B), block(kAccThreads);
    uint32_t *seq_counters = reinterpret_cast<uint32_t *>(ws);
    uint32_t *row_counters = reinterpret_cast<uint32_t *>(ws + plan.row_counters_off);
    unsigned long long *row_keys = reinterpret_cast<unsigned long long *>(ws + plan.keys_off);
    const uint32_t inv_l = ((1u << 20) + (uint32_t)L - 1) / (uint32_t)L;      // e / L = e * inv_l >> 20 for e < RD_MAX_N
    static_assert(RD_MAX_N * RD_MAX_N <= 1 << 20, "error of the reciprocal times e below 1 / L");
#define RD_ACCEPT_LAUNCH_(U, SPEC)                                                                            \
    hipLaunchKernelGGL((rd_accept_kernel<U, SPEC>), grid, block, 0, stream, logits, beams, unpack_index,       \
                       n_packed, root_token, W, L, V, plan.chunks, plan.chunk_len, inv_l, argmax_out, n_accept,       \
                       best_beam, best_len, next_token, accepted_idx, seq_counters, row_counters, row_keys)
#define RD_ACCEPT_LAUNCH(U)                                 \
    do {                                                    \
        if (plan.speculate) RD_ACCEPT_LAUNCH_(U, true);     \
        else RD_ACCEPT_LAUNCH_(U, false);                   \
    } while (0)
    switch (plan.loads) {
    case 1: RD_ACCEPT_LAUNCH(1); break;
    case 2: RD_ACCEPT_LAUNCH(2); break;
    case 4: RD_ACCEPT_LAUNCH(4); break;
    case 8: RD_ACCEPT_LAUNCH(8); break;
    case 16: RD_ACCEPT_LAUNCH_(16, false); break;
    default: RD_ACCEPT_LAUNCH_(32, false); break;
    }
#undef RD_ACCEPT_LAUNCH
#undef RD_ACCEPT_LAUNCH_
    return rd_check_launch();
}

extern "C" int rd_accept(const float *logits, const int32_t *beams, const int32_t *unpack_index,
                         const int32_t *n_packed, const int32_t *root_token,
                         int B, int W, int L, int V,
                         int32_t *argmax_out, int32_t *n_accept, int32_t *best_beam,
                         int32_t *best_len, int32_t *next_token, int32_t *accepted_idx,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    AccPlan plan;
    const int st = accept_check(logits, beams, unpack_index, n_packed, B, W, L, V, argmax_out, n_accept, best_beam,
                                best_len, next_token, accepted_idx, &plan);
    if (st != RD_OK) return st;
    if (!workspace || !rd_aligned(workspace, 256) || workspace_bytes < plan.total_bytes) return RD_ERR_WORKSPACE;
    return accept_launch(plan, logits, beams, unpack_index, n_packed, root_token, B, W, L, V, argmax_out, n_accept,
                         best_beam, best_len, next_token, accepted_idx, static_cast<unsigned char *>(workspace),
                         (hipStream_t)stream);
}

// ---- rd_accept_static: the same call for callers that cannot allocate ---------------------------
// The counters and row keys live in a file-scope device array instead of a caller-provided
// workspace.  Every device that loads the library holds its own copy of the array at its own
// address until the process ends; the address is looked up once per device, with that device
// current, and only that address (never the array's name, which in host code is a stand-in and
// not a device address) is handed to kernels.
static __device__ __align__(256) unsigned char scratch[RD_ACCEPT_STATIC_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<unsigned char *> g_scratch_ptr[kMaxDevices];     // device address of `scratch`, per device, once known

int static_scratch(unsigned char **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return RD_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return RD_ERR_UNSUPPORTED;
    unsigned char *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        void *sym = nullptr;
        if (hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)) != hipSuccess || sym == nullptr) return RD_ERR_HIP;
        p = static_cast<unsigned char *>(sym);
        g_scratch_ptr[dev].store(p, std::memory_order_release);     // two threads racing here store the same address
    }
    *out = p;
    return RD_OK;
}

// Zeroes n_vec 16-byte vectors.  A kernel rather than a memset so that the call stays safe to
// capture into a HIP graph.
__global__ __launch_bounds__(256) void rd_clear_kernel(uint4 *p, size_t n_vec)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_vec) p[i] = make_uint4(0, 0, 0, 0);
}

}  // namespace

extern "C" int rd_accept_static(const float *logits, const int32_t *beams, const int32_t *unpack_index,
                                const int32_t *n_packed, const int32_t *root_token,
                                int B, int W, int L, int V,
                                int32_t *argmax_out, int32_t *n_accept, int32_t *best_beam,
                                int32_t *best_len, int32_t *next_token, int32_t *accepted_idx, void *stream)
{
    AccPlan plan;
    const int st = accept_check(logits, beams, unpack_index, n_packed, B, W, L, V, argmax_out, n_accept, best_beam,
                                best_len, next_token, accepted_idx, &plan);
    if (st != RD_OK) return st;
    if (plan.total_bytes > (size_t)RD_ACCEPT_STATIC_BYTES) return RD_ERR_SCRATCH_LIMIT;
    unsigned char *ws = nullptr;
    const int sp = static_scratch(&ws);
    if (sp != RD_OK) return sp;
    // The array keeps whatever the last call on this device left (normally zeros, but a call that was
    // aborted, or one of another shape that failed, may leave anything): clear the part this call uses.
    const size_t n_vec = plan.total_bytes / 16;                     // every section is a multiple of 256 bytes
    hipLaunchKernelGGL(rd_clear_kernel, dim3((unsigned)((n_vec + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<uint4 *>(ws), n_vec);
    const int cl = rd_check_launch();
    if (cl != RD_OK) return cl;
    return accept_launch(plan, logits, beams, unpack_index, n_packed, root_token, B, W, L, V, argmax_out, n_accept,
                         best_beam, best_len, next_token, accepted_idx, ws, (hipStream_t)stream);
}
