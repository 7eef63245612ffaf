// rd_accept_sample: acceptance by rejection sampling (Sec. 3.4's sampling mode; speculative
// sampling applied to every candidate on the packed tree) for gfx950, two launches.
//
// Launch 1 (the HBM stream): grid (chunks, N, B); a workgroup reduces one chunk of 4096 entries of a
// valid row of the LLM's logits (scaled by 1/temperature) and of the draft model's logits to
// (maximum, sum of exp(x - maximum)) each and stores the two pairs in the workspace.  Every wave finds by itself which
// draft row belongs to the slot, the 16-byte loads of a row are in flight together, and the waves meet
// once.  Rows of slots at the last position carry no draft distribution and their draft half is skipped.  No
// atomics, no counters: the partials are combined in a fixed order by launch 2, so results do not depend on timing.  It also
// clears the words in which launch 2 hands over its chunks' totals.
// Launch 2 (grid: chunks of 4096 vocabulary entries x sequences, 256 threads).  Every workgroup of a
// sequence repeats the small part: log-sum-exps of the rows from the partials; one thread per
// candidate token gathers the two logits of its token under its parent slot and decides
// u < min(1, p/q); one thread per candidate counts its accepted prefix; the best candidate is the
// longest (smallest index among equals).  The token that follows is drawn by inverting a cumulative
// distribution with the caller's uniform number.  One compute unit alone needs ~10 us for the 2 x V
// exponentials of a residual max(0, p - q), so that pass is spread: each workgroup sums the residual
// weights of its own chunk, stores the total and signals; the last one to arrive adds the totals in
// chunk order, finds the chunk in which the running total crosses the target, recomputes that
// chunk's weights and takes, by a block-wide prefix scan, the first token of positive weight whose
// cumulative weight exceeds the target.  After a fully accepted candidate the weights are p itself,
// whose chunk totals follow from launch 1's partials: workgroup 0 goes straight to the last step.
// Both launches are chains of memory round trips (0.6-1 us each), so what bounds them is the number of loads that wait
// for another -- the partials of all rows and chunks, the tokens and the gathered logits are fetched side by side, and
// the totals travel as write-through stores (a device-scope fence writes back the XCD's L2) that nobody waits for before
// arriving -- and, in launch 2, a lone wave's instructions (1.7 ns each): tests and accepted prefixes are ballots.  us a call
// against tests through LDS and atomics, barriers that waited for stores and arrivals that waited for totals: 8 sequences of
// 8 x 5 tokens, V = 32000 21.9 -> 19.2, one 14.1 -> 12.1, 70 x 5 25.4 -> 21.9, 16 of 16 x 5 39.0 -> 36.5.
#include "rd_internal.h"
#include <math.h>

RD_TRACE_DEFINE(rd_debug_set_trace_sample)

namespace {

constexpr int kLseThreads = 256;
constexpr int kLseChunk = 4096;              // entries per workgroup of launch 1: 4 x 16 bytes per thread and array
constexpr int kSelThreads = 256;
constexpr int kSelPer = 16;                  // consecutive entries per thread of launch 2
constexpr int kSelChunk = kSelPer * kSelThreads;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kMaxSelChunks = 256;           // V <= 1 Mi entries
constexpr int kTokens = (RD_MAX_N + kSelThreads - 1) / kSelThreads;      // per thread
static_assert(kSelChunk == kLseChunk, "launch 2 takes the chunk totals of p from launch 1's partials");

// Entries v .. v+3 of a row, -inf past the end (weight 0, neutral for the maximum).  VEC: rows of four entries and
// more, 16-byte loads, in their places if ORDERED; else scalar loads.
template <bool VEC, bool ORDERED>
__device__ __forceinline__ float4 load4(const float *row, int v, int V)
{
    if constexpr (VEC) {
        return ORDERED ? rd::row4(row, v, V) : rd::row4_set(row, v, V);
    } else {
        const float x = row[min(v, V - 1)], y = row[min(v + 1, V - 1)], z = row[min(v + 2, V - 1)], w = row[min(v + 3, V - 1)];
        return make_float4(v < V ? x : -INFINITY, v + 1 < V ? y : -INFINITY, v + 2 < V ? z : -INFINITY, v + 3 < V ? w : -INFINITY);
    }
}

// (maximum, sum exp(x*scale - maximum)) of 16 values per lane over the wave
__device__ __forceinline__ float2 wave_max_sum(const float4 (&x)[4], float scale)
{
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(fmaxf(fmaxf(x[u].x, x[u].y), fmaxf(x[u].z, x[u].w)) * scale, m);
    m = rd::wave_reduce_max(m);
    float s = 0.f;
    const float ms = m > -INFINITY ? m : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        s += __expf(x[u].x * scale - ms) + __expf(x[u].y * scale - ms) + __expf(x[u].z * scale - ms) + __expf(x[u].w * scale - ms);
    return make_float2(m, rd::wave_reduce_sum(s));
}
// the same over waves
__device__ __forceinline__ float2 merge_max_sum(float2 a, float2 b)
{
    const float m = fmaxf(a.x, b.x), ms = m > -INFINITY ? m : 0.f;
    return make_float2(m, a.y * __expf(a.x - ms) + b.y * __expf(b.x - ms));
}

// The draft model's logits of the distribution after candidate w's token j (which sits in packed
// slot `slot`): row `slot` of the packed layout [B][N][V], or, in the layout the beam search records
// ([L-1][rows_per_step][V] plus step_row [B][W][L-1]), row step_row[b][w][j] of step j.
__device__ __forceinline__ const float *draft_row_ptr(const float *draft_logits, const int32_t *step_row, int rows_per_step,
                                                      int b, int w, int j, int slot, int W, int L, int V)
{
    if (step_row == nullptr) return draft_logits + ((size_t)b * W * L + slot) * V;
    const int r = min(max(step_row[((size_t)b * W + w) * (L - 1) + j], 0), rows_per_step - 1);
    return draft_logits + ((size_t)j * rows_per_step + r) * V;
}

template <bool VEC>
__global__ __launch_bounds__(kLseThreads) void rd_lse_chunk_kernel(
    const float *__restrict__ logits, const float *__restrict__ draft_logits, const int32_t *__restrict__ step_row,
    int rows_per_step, const int32_t *__restrict__ unpack_index,
    const int32_t *__restrict__ n_packed, int W, int L, int V, int chunks, float inv_t, float4 *__restrict__ part,
    float *__restrict__ chunk_totals /*[B][chunks]*/)
{
    constexpr int kWaves = kLseThreads / 64;
    __shared__ float4 s_red[kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x, p = blockIdx.y, b = blockIdx.z;
    const int N = W * L;
    // which (candidate, position) this slot holds: the first entry of unpack_index that names it.  Every wave looks
    // through all entries while they are few; else each thread takes some and the waves meet.
    constexpr int kWaveScan = 2, kTok = (RD_MAX_N + kLseThreads - 1) / kLseThreads;
    __shared__ int s_owner[kWaves];
    const bool by_wave = N <= 64 * kWaveScan;               // uniform
    const int first = by_wave ? lane : tid, stride = by_wave ? 64 : kLseThreads;
    int slot[kWaveScan];
    static_assert(kTok <= kWaveScan, "entries per thread");
#pragma unroll
    for (int i = 0; i < kWaveScan; ++i) slot[i] = unpack_index[(size_t)b * N + min(i * stride + first, N - 1)];
    int P = n_packed[b];
    P = P < 1 ? 1 : (P > N ? N : P);
    if (p >= P) return;
    const size_t rowid = (size_t)b * N + p;
    const float *zp = logits + rowid * V;
    const int v0 = chunk * kLseChunk;
    float4 xp[4], xq[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) xp[u] = load4<VEC, false>(zp, v0 + (u * kLseThreads + tid) * 4, V);
    int owner = 0x7fffffff;
#pragma unroll
    for (int i = kWaveScan - 1; i >= 0; --i) {
        const unsigned long long hit = __ballot(slot[i] == p && i * stride + first < N);
        if (hit) owner = i * stride + (by_wave ? 0 : wave * 64) + __ffsll((long long)hit) - 1;
    }
    if (!by_wave) {
        if (lane == 0) s_owner[wave] = owner;
        rd_lds_barrier();
        owner = min(min(s_owner[0], s_owner[1]), min(s_owner[2], s_owner[3]));
    }
    owner = __builtin_amdgcn_readfirstlane(owner);
    // The LLM's row is reduced before the draft model's is fetched (the empty asm keeps that order): with both in flight
    // the launch takes longer, 9.4 against 8.6 us at B=4, W=48, L=3, V=20000.
    float2 a = wave_max_sum(xp, inv_t);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" :: "v"(a.x), "v"(a.y) : "memory");
    const int ow = owner / L, oj = owner - ow * L;
    const bool draft = owner != 0x7fffffff && oj < L - 1;   // uniform: not at the last position, a draft row exists
    if (draft) {
        const float *zq = draft_row_ptr(draft_logits, step_row, rows_per_step, b, ow, oj, p, W, L, V);
#pragma unroll
        for (int u = 0; u < 4; ++u) xq[u] = load4<VEC, false>(zq, v0 + (u * kLseThreads + tid) * 4, V);
    }
    float2 c = make_float2(0.f, 1.f / kWaves);
    if (draft) c = wave_max_sum(xq, 1.0f);
    if (lane == 0) s_red[wave] = make_float4(a.x, a.y, c.x, c.y);
    __syncthreads();
    if (tid == 0) {
        a = make_float2(s_red[0].x, s_red[0].y);
        c = make_float2(s_red[0].z, s_red[0].w);
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            a = merge_max_sum(a, make_float2(s_red[w].x, s_red[w].y));
            c = merge_max_sum(c, make_float2(s_red[w].z, s_red[w].w));
        }
        part[rowid * chunks + chunk] = make_float4(a.x, a.y, c.x, c.y);
        if (p == 0) chunk_totals[(size_t)b * chunks + chunk] = 0.f;      // launch 2 waits until it is not
    }
}

// weight of entry v in the distribution the next token is drawn from
__device__ __forceinline__ float weight(float zp, float zq, float inv_t, float lse_p, float lse_q, bool residual)
{
    const float p = __expf(zp * inv_t - lse_p);             // exp(-inf) = 0 past the end of the row
    if (!residual) return p;
    return fmaxf(p - __expf(zq - lse_q), 0.f);
}

// Exclusive prefix sums of one value per thread over the workgroup, in thread order; `total` gets the
// workgroup's sum (the same bits in every thread).
__device__ __forceinline__ float block_exclusive_scan(float x, float *s_wave, float &total)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    rd_lds_barrier();                                        // s_wave free again
    if (lane == 63) s_wave[wave] = incl;
    rd_lds_barrier();
    float before = 0.f, all = 0.f;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        const float t = s_wave[w];
        if (w < wave) before += t;
        all += t;
    }
    total = all;
    return before + (incl - x);
}

// The 16 consecutive weights of this thread in chunk `chunk` of the row; returns their sum.
template <bool VEC>
__device__ __forceinline__ float chunk_weights(const float *zp, const float *zq, int chunk, int V, float inv_t,
                                               float lse_p, float lse_q, bool residual, float (&w)[kSelPer])
{
    const int v0 = chunk * kSelChunk + threadIdx.x * kSelPer;
    const float *zr = residual ? zq : zp;                   // no draft row to read when drawing from p (value unused)
    float4 a[kSelPer / 4], q[kSelPer / 4];
#pragma unroll
    for (int i = 0; i < kSelPer / 4; ++i) a[i] = load4<VEC, true>(zp, v0 + 4 * i, V);
#pragma unroll
    for (int i = 0; i < kSelPer / 4; ++i) q[i] = load4<VEC, true>(zr, v0 + 4 * i, V);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < kSelPer / 4; ++i) {
        w[4 * i + 0] = weight(a[i].x, q[i].x, inv_t, lse_p, lse_q, residual);
        w[4 * i + 1] = weight(a[i].y, q[i].y, inv_t, lse_p, lse_q, residual);
        w[4 * i + 2] = weight(a[i].z, q[i].z, inv_t, lse_p, lse_q, residual);
        w[4 * i + 3] = weight(a[i].w, q[i].w, inv_t, lse_p, lse_q, residual);
        sum += ((w[4 * i] + w[4 * i + 1]) + w[4 * i + 2]) + w[4 * i + 3];
    }
    return sum;
}

template <bool VEC>
__global__ __launch_bounds__(kSelThreads) void rd_accept_sample_kernel(
    const float *__restrict__ logits, const float *__restrict__ draft_logits, const int32_t *__restrict__ step_row,
    int rows_per_step, const int32_t *__restrict__ beams,
    const int32_t *__restrict__ unpack_index, const int32_t *__restrict__ n_packed,
    const int32_t *__restrict__ root_token, const float *__restrict__ u_accept, const float *__restrict__ u_next,
    int W, int L, uint32_t inv_l /* e / L = e * inv_l >> 20 */, int V, int chunks, float inv_t, const float4 *__restrict__ part,
    float *chunk_totals /*[B][chunks]*/, uint32_t *counters /*[B]*/,
    int32_t *__restrict__ n_accept, int32_t *__restrict__ best_beam, int32_t *__restrict__ best_len,
    int32_t *__restrict__ next_token, int32_t *__restrict__ accepted_idx)
{
    __shared__ float s_lse_p[RD_MAX_N], s_lse_q[RD_MAX_N];
    __shared__ int s_slot[RD_MAX_N];
    __shared__ unsigned long long s_ok[kTokens * kSelWaves];
    __shared__ int s_best[2], s_pick[kSelWaves], s_lastpos[kSelWaves];
    __shared__ uint32_t s_last;
    __shared__ float s_wave[kSelWaves];
    __shared__ int s_ci, s_residual;
    __shared__ float s_base, s_target;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int N = W * L;
    int P = n_packed[b];
    P = P < 1 ? 1 : (P > N ? N : P);
    const int my_root = root_token ? root_token[b] : 0;
    const float u_draw = u_next[b];
    RD_TR(0);

    // ---- every workgroup of the sequence: log-sum-exps, rejection tests, best candidate -------------------
    // candidate tokens: at most two per thread; slot of a token and of its parent, and (where it has one) the
    // draft distribution it was drawn from, all fetched before anything waits
    constexpr int kTok = kTokens;
    int tx[kTok], ts[kTok], tc[kTok], tr[kTok], tj[kTok];    // (tj: position in the candidate)
    const bool has_row = step_row != nullptr && L > 1;
    // Up to 64 tokens every wave tests all of them, so that no barrier stands behind the tests.
    const bool by_wave = N <= 64;                           // uniform
    const int token0 = by_wave ? lane : tid;
    auto over_l = [&](int e) __attribute__((always_inline)) { return (int)((uint32_t)e * inv_l >> 20); };     // e / L
#pragma unroll
    for (int k = 0; k < kTok; ++k) {
        const int e = min(k * kSelThreads + token0, N - 1), ep = max(e - 1, 0), j = tj[k] = e - over_l(e) * L;
        tx[k] = beams[(size_t)b * N + e];
        tc[k] = unpack_index[(size_t)b * N + e];
        ts[k] = unpack_index[(size_t)b * N + ep];
        tr[k] = *(has_row ? step_row + ((size_t)b * W + over_l(e)) * (L - 1) + max(j - 1, 0) : n_packed);   // (no branch around a load)
    }
    // Partials: a group of G lanes (a power of two) takes a row, one or more chunks per lane; up to kRowsAhead rows per
    // lane group have their loads in flight together, the first of them beside the logits gathered below.  Rows of
    // padding slots are read and ignored.
    constexpr int kRowsAhead = 4;
    int G = 1;
    while (G < chunks && G < 64) G <<= 1;
    const int rows_per = kSelThreads / G, gl = tid & (G - 1), gr = tid / G;
    float4 v[kRowsAhead];
    auto load_rows = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kRowsAhead; ++k) {
            const int r = min(r0 + k * rows_per + gr, N - 1);
            v[k] = part[((size_t)b * N + r) * chunks + min(gl, chunks - 1)];
        }
    };
    load_rows(0);
    // the logits of the candidate tokens under their parents
    float zp_t[kTok], zq_t[kTok], u_t[kTok];
#pragma unroll
    for (int k = 0; k < kTok; ++k) {
        const int e = min(k * kSelThreads + token0, N - 1), j = max(tj[k], 1);
        const int x = min(max(tx[k], 0), V - 1);
        tc[k] = min(max(tc[k], 0), N - 1);
        ts[k] = min(max(ts[k], 0), N - 1);
        const int s = tj[k] == 0 ? 0 : ts[k];
        const size_t qrow = has_row ? (size_t)(j - 1) * rows_per_step + min(max(tr[k], 0), rows_per_step - 1) : (size_t)b * N + s;
        zp_t[k] = L > 1 ? logits[((size_t)b * N + s) * V + x] : 0.f;
        zq_t[k] = L > 1 ? draft_logits[qrow * V + x] : 0.f;
        u_t[k] = u_accept[(size_t)b * N + tc[k]];
        if (k * kSelThreads + token0 < N) s_slot[e] = tc[k];
    }
    auto larger = [](float a, float c) __attribute__((always_inline)) { return fmaxf(a, c); };
    auto plus = [](float a, float c) __attribute__((always_inline)) { return a + c; };
    auto reduce_rows = [&](int r0, const float4 *rows) __attribute__((always_inline)) {
        constexpr int K = kRowsAhead / 2;
        float mp[K], mq[K], sp[K], sq[K];
        float4 x[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] = gl < chunks ? rows[k] : make_float4(-INFINITY, 0.f, -INFINITY, 0.f);
            for (int c = gl + G; c < chunks; c += G) {      // more than 64 chunks
                const float4 y = part[((size_t)b * N + min(r0 + k * rows_per + gr, N - 1)) * chunks + c];
                const float2 p2 = merge_max_sum(make_float2(x[k].x, x[k].y), make_float2(y.x, y.y));
                const float2 q2 = merge_max_sum(make_float2(x[k].z, x[k].w), make_float2(y.z, y.w));
                x[k] = make_float4(p2.x, p2.y, q2.x, q2.y);
            }
            mp[k] = x[k].x;
            mq[k] = x[k].z;
        }
        rd::group_reduce(mp, G, larger);
        rd::group_reduce(mq, G, larger);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sp[k] = x[k].y * __expf(x[k].x - (mp[k] > -INFINITY ? mp[k] : 0.f));
            sq[k] = x[k].w * __expf(x[k].z - (mq[k] > -INFINITY ? mq[k] : 0.f));
        }
        rd::group_reduce(sp, G, plus);
        rd::group_reduce(sq, G, plus);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int r = r0 + k * rows_per + gr;
            if (gl == 0 && r < P) {
                s_lse_p[r] = mp[k] + __logf(sp[k]);
                s_lse_q[r] = mq[k] + __logf(sq[k]);
            }
        }
    };
    for (int r0 = 0;;) {
        reduce_rows(r0, v);
        if (r0 + kRowsAhead / 2 * rows_per < P) reduce_rows(r0 + kRowsAhead / 2 * rows_per, v + kRowsAhead / 2);     // uniform
        r0 += kRowsAhead * rows_per;
        if (r0 >= P) break;                                 // uniform
        load_rows(r0);
    }
    rd_lds_barrier();
    RD_TR(1);

    // the rejection test of token (w, j), j >= 1, a bit each
    uint64_t bits[kTok];
#pragma unroll
    for (int k = 0; k < kTok; ++k) {
        const int e = k * kSelThreads + token0, x = tx[k];
        bool ok = false;
        if (e < N) {
            if (tj[k] == 0) {
                ok = (root_token == nullptr) || (x == my_root);
            } else {
                const float lp = zp_t[k] * inv_t - s_lse_p[ts[k]], lq = zq_t[k] - s_lse_q[ts[k]];
                ok = x >= 0 && x < V && u_t[k] < fminf(__expf(lp - lq), 1.0f);
            }
        }
        bits[k] = __ballot(ok);
    }
    RD_TR(2);

    // one thread per candidate: length of the accepted prefix; best = longest, then smallest index
    static_assert(RD_MAX_W <= 128 && RD_MAX_N < (1 << 15), "candidates: two waves, index in 8 bits");
    int key;
    if (by_wave) {
        const int len = rd::accepted_run(bits[0], min(lane * L, 63), L);
        if (chunk == 0 && tid < W) n_accept[(size_t)b * W + tid] = len;
        key = rd::wave_reduce_max_i(lane < W ? (len << 8) | (255 - lane) : 0);
    } else {
#pragma unroll
        for (int k = 0; k < kTok; ++k)
            if (lane == 0) s_ok[k * kSelWaves + wave] = bits[k];
        rd_lds_barrier();
        int len = 0;
        if (tid < W) {
            len = rd::accepted_run(s_ok, tid * L, L);
            if (chunk == 0) n_accept[(size_t)b * W + tid] = len;
        }
        if (wave < 2) {
            const int most = rd::wave_reduce_max_i(tid < W ? (len << 8) | (255 - tid) : 0);
            if (lane == 0) s_best[wave] = most;
        }
        rd_lds_barrier();
        key = max(s_best[0], s_best[1]);
    }
    RD_TR(3);
    const int bl = key >> 8, bw = 255 - (key & 255);
    if (chunk == 0) {
        for (int t = tid; t < L; t += kSelThreads) accepted_idx[(size_t)b * L + t] = (t < bl) ? s_slot[bw * L + t] : -1;
        if (tid == 0) { best_beam[b] = bw; best_len[b] = bl; }
    }
    if (bl == 0) {                                          // the first token was refuted: nothing to draw
        if (chunk == 0 && tid == 0) next_token[b] = my_root;
        return;
    }

    // ---- the next token: inverse CDF of p (whole candidate accepted) or of the residual -------------------
    const int s = s_slot[bw * L + bl - 1];
    const float *zp = logits + ((size_t)b * N + s) * V;
    // (not read when the candidate was accepted whole)
    const float *zq = bl < L ? draft_row_ptr(draft_logits, step_row, rows_per_step, b, bw, bl - 1, s, W, L, V) : zp;
    const float lse_p = s_lse_p[s], lse_q = s_lse_q[s];
    const float4 *prow = part + ((size_t)b * N + s) * chunks;
    bool residual = bl < L;
    float w[kSelPer];
    if (residual) {
        // this workgroup's chunk of the residual: total -> workspace, then find out who is last
        float t = chunk_weights<VEC>(zp, zq, chunk, V, inv_t, lse_p, lse_q, true, w);
        t = rd::wave_reduce_sum(t);
        if (lane == 0) s_wave[wave] = t;
        rd_lds_barrier();
        if (tid == 0) {
            // A total is never negative: with its sign set it cannot be taken for the word that launch 1 cleared, and whoever
            // arrives last reads it until it is there (rd::poll).  (It was issued before the arrival: nothing waits for it here.)
            const float total = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
            rd::st_dev(chunk_totals + (size_t)b * chunks + chunk, __uint_as_float(__float_as_uint(total) | 0x80000000u));
            const uint32_t prev = __hip_atomic_fetch_add(counters + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = (prev + 1u == (uint32_t)chunks) ? 1u : 0u;
        }
        rd_lds_barrier();
        if (!s_last) return;
        if (tid == 0) counters[b] = 0;                      // ready for the next call
    } else if (chunk != 0) {
        return;
    }
    RD_TR(4);
    // Running totals of the chunks in chunk order, by the first wave: lane l holds chunks per*l .. per*l + per - 1.
    // The chunk in which the running total crosses the target; if rounding leaves none, the last that holds any weight.
    if (wave == 0) {
        const int per = (chunks + 63) / 64;
        float mine[kMaxSelChunks / 64], sum = 0.f;
        bool any = false;
        for (int attempt = 0; attempt < 2; ++attempt) {     // once more if p == q everywhere: draw from p
            sum = 0.f;
#pragma unroll
            for (int k = 0; k < kMaxSelChunks / 64; ++k) {
                const int i = min(lane * per + k, chunks - 1);
                mine[k] = 0.f;
                if (k < per) {
                    float t;
                    if (residual) {
                        const uint32_t u = rd::poll([&]() { return __float_as_uint(rd::ld_dev(chunk_totals + (size_t)b * chunks + i)); },
                                                    [](uint32_t x) { return (x & 0x80000000u) != 0; });
                        t = __uint_as_float(u & 0x7fffffffu);
                    } else {
                        t = prow[i].y * __expf(prow[i].x - lse_p);      // totals of p from launch 1's partials
                    }
                    if (lane * per + k < chunks) mine[k] = t;
                }
                sum += mine[k];
            }
            any = __ballot(sum > 0.f) != 0;
            if (any || !residual) break;
            residual = false;
        }
        float incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const float o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        const float target = u_draw * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(incl), 63));
        float run = incl - sum, base = 0.f;
        int ci = 0x7fffffff, lastc = -1;
#pragma unroll
        for (int k = 0; k < kMaxSelChunks / 64; ++k) {
            if (mine[k] > 0.f) lastc = lane * per + k;
            const float next = run + mine[k];
            if (ci == 0x7fffffff && mine[k] > 0.f && target < next) { ci = lane * per + k; base = run; }
            run = next;
        }
        const unsigned long long cross = __ballot(ci != 0x7fffffff), held = __ballot(lastc >= 0);
        if (cross) {
            const int w0 = __ffsll((long long)cross) - 1;
            ci = __builtin_amdgcn_readlane(ci, w0);
            base = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(base), w0));
        } else {
            ci = held ? __builtin_amdgcn_readlane(lastc, 63 - __clzll((long long)held)) : 0;
            base = 0.f;
        }
        if (lane == 0) { s_ci = ci; s_base = base; s_target = target; s_residual = residual ? 1 : 0; }
    }
    rd_lds_barrier();
    const int ci = s_ci;
    const float base = s_base, target = s_target;
    residual = s_residual != 0;
    // cumulative weights inside the chunk, in token order.  The scan sums in another order than the
    // chunk totals did, so its last value may fall short of the target by rounding: then the chunk's
    // last token of positive weight is the one.
    const float tsum = chunk_weights<VEC>(zp, zq, ci, V, inv_t, lse_p, lse_q, residual, w);
    float chunk_total;
    float cum = base + block_exclusive_scan(tsum, s_wave, chunk_total), upto[kSelPer];
#pragma unroll
    for (int k = 0; k < kSelPer; ++k) upto[k] = cum += w[k];
    const int v0 = ci * kSelChunk + tid * kSelPer;
    int pick = -1;
#pragma unroll
    for (int k = kSelPer - 1; k >= 0; --k) pick = w[k] > 0.f && upto[k] > target ? v0 + k : pick;
    // (tokens ascend with the threads)
    const uint64_t found = __ballot(pick >= 0);
    const int first = found ? __builtin_amdgcn_readlane(pick, __ffsll((long long)found) - 1) : 0x7fffffff;
    if (lane == 0) s_pick[wave] = first;
    rd_lds_barrier();
    RD_TR(5);
    int tok = min(min(s_pick[0], s_pick[1]), min(s_pick[2], s_pick[3]));
    if (tok == 0x7fffffff) {                                // rounding left no crossing: the last token of positive weight
        int lastpos = -1;
#pragma unroll
        for (int k = 0; k < kSelPer; ++k) lastpos = w[k] > 0.f ? v0 + k : lastpos;
        const uint64_t held = __ballot(lastpos >= 0);
        if (lane == 0) s_lastpos[wave] = held ? __builtin_amdgcn_readlane(lastpos, 63 - __clzll((long long)held)) : -1;
        rd_lds_barrier();
        tok = max(max(s_lastpos[0], s_lastpos[1]), max(s_lastpos[2], s_lastpos[3]));
    }
    if (tid == 0) {
        if (tok < 0) tok = 0;
        next_token[b] = tok;
    }
}

struct SamplePlan {
    int chunks;
    size_t totals_off, part_off;         // byte offsets in the workspace (arrival counters at 0)
    size_t total_bytes;
};

SamplePlan sample_plan(int B, int N, int V)
{
    SamplePlan p;
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    p.chunks = (V + kLseChunk - 1) / kLseChunk;
    p.totals_off = up((size_t)B * sizeof(uint32_t));
    p.part_off = p.totals_off + up((size_t)B * p.chunks * sizeof(float));
    p.total_bytes = p.part_off + up((size_t)B * N * p.chunks * sizeof(float4));
    return p;
}

}  // namespace

extern "C" size_t rd_accept_sample_workspace(int B, int W, int L, int V)
{
    if (rd_check_beam_shape(B, W, L) != RD_OK || V <= 0 || V > kMaxSelChunks * kSelChunk) return 0;
    return sample_plan(B, W * L, V).total_bytes;
}

extern "C" int rd_accept_sample(const float *logits, const float *draft_logits, const int32_t *draft_step_row,
                                int draft_rows_per_step, const int32_t *beams, const int32_t *unpack_index, const int32_t *n_packed, const int32_t *root_token,
                                const float *u_accept, const float *u_next, float temperature,
                                int B, int W, int L, int V,
                                int32_t *n_accept, int32_t *best_beam, int32_t *best_len, int32_t *next_token,
                                int32_t *accepted_idx, void *workspace, size_t workspace_bytes, void *stream)
{
    const int st = rd_check_beam_shape(B, W, L);
    if (st != RD_OK) return st;
    if (V <= 0 || !(temperature > 0.f) || !isfinite(temperature)) return RD_ERR_INVALID_ARG;
    if (B > 65535 || V > kMaxSelChunks * kSelChunk) return RD_ERR_UNSUPPORTED;
    if (!logits || !draft_logits || !beams || !unpack_index || !n_packed || !u_accept || !u_next || !n_accept ||
        !best_beam || !best_len || !next_token || !accepted_idx)
        return RD_ERR_INVALID_ARG;
    if (!rd_aligned(logits, 16) || !rd_aligned(draft_logits, 16)) return RD_ERR_INVALID_ARG;
    if (draft_step_row != nullptr && draft_rows_per_step <= 0) return RD_ERR_INVALID_ARG;
    const int N = W * L;
    const SamplePlan plan = sample_plan(B, N, V);
    if (!workspace || !rd_aligned(workspace, 256) || workspace_bytes < plan.total_bytes) return RD_ERR_WORKSPACE;
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    uint32_t *counters = reinterpret_cast<uint32_t *>(ws);
    float *chunk_totals = reinterpret_cast<float *>(ws + plan.totals_off);
    float4 *part = reinterpret_cast<float4 *>(ws + plan.part_off);
    const float inv_t = 1.0f / temperature;
    hipStream_t s = (hipStream_t)stream;
    const bool vec = V >= 4;
    hipLaunchKernelGGL(vec ? rd_lse_chunk_kernel<true> : rd_lse_chunk_kernel<false>, dim3(plan.chunks, N, B),
                       dim3(kLseThreads), 0, s, logits, draft_logits, draft_step_row, draft_rows_per_step, unpack_index, n_packed, W, L, V,
                       plan.chunks, inv_t, part, chunk_totals);
    if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
    hipLaunchKernelGGL(vec ? rd_accept_sample_kernel<true> : rd_accept_sample_kernel<false>, dim3(plan.chunks, B),
                       dim3(kSelThreads), 0, s, logits, draft_logits, draft_step_row, draft_rows_per_step, beams, unpack_index, n_packed,
                       root_token, u_accept,
                       u_next, W, L, ((1u << 20) + (uint32_t)L - 1) / (uint32_t)L, V, plan.chunks, inv_t, part, chunk_totals, counters, n_accept, best_beam, best_len,
                       next_token, accepted_idx);
    return rd_check_launch();
}
