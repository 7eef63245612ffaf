// rd_dedup: dynamic tree attention construction (Sec. 3.3, App. A.1) for gfx950.
//
// Up to 64 tokens: rd_dedup_wave_kernel below; more, in candidates of up to 64: rd_dedup_waves_kernel.  Longer ones (five at most):
// One workgroup per sequence (more where the dense mask is asked for), everything in LDS, data-parallel phases
// separated by barriers (the whole input is a few hundred bytes; what costs time is dependent latency, so no phase
// is a serial walk over positions):
//   A  stage the W x L candidates; owner[i][j] = i.
//   B  one thread per ordered pair (i, k < i): walk their common prefix and lower owner[i][j]
//      to k (LDS atomic min) for every j inside it.  Afterwards owner[i][j] is the smallest
//      candidate sharing i's first j+1 tokens, i.e. prefix_tree — the equal-length property
//      the paper exploits, with no trie and no data-dependent pointer chasing.
//   C  a token is kept iff owner == i; kept tokens of a candidate are a suffix of its row, so
//      each row's first kept position and a prefix sum of the kept counts give every row
//      its first packed slot (row-major slot order).
//   D  one thread per token: slot of its owner's copy -> unpack_index.
//   E  one thread per kept token: packed token, parent, position id, and the mask row as the
//      OR of the slots on its path.
//   F  paddings, the bit-packed and the dense mask, with coalesced stores.
#include "rd_internal.h"

RD_TRACE_DEFINE(rd_debug_set_trace_dedup)

namespace {

constexpr int kDedupThreads = 384;                 // of rd_dedup_kernel: one thread per token
// Rows of the dense mask per workgroup; every workgroup repeats the construction.  us by 16 / 32 / 48 / 64 rows: N = 80, 16 sequences
// 3.81 / 3.77 / 3.77 / 3.85, N = 150 4.43 / 4.59 / 4.83 / 4.99, N = 350 7.25 / 7.62 / 8.04 / 8.45 and 24 sequences of it 9.39 / 8.82 / 8.73 / 9.09,
// 60 sequences of N = 240 10.25 / 6.52 / 6.71 / 6.60.
constexpr int kMaskRows = 32;
constexpr int kMaskWords = (RD_MAX_N + 63) / 64;
constexpr int kMaskWaves = 8;                      // at least, where the dense mask is written
constexpr int kMaxTokenWaves = 11;                 // of rd_dedup_waves_kernel: 33 positions, one candidate to a wave

__global__ __launch_bounds__(kDedupThreads) void rd_dedup_kernel(
    const int32_t *__restrict__ beams, const int32_t *__restrict__ ctx_len, int W, int L,
    int32_t *__restrict__ prefix_tree, int32_t *__restrict__ packed_tokens,
    int32_t *__restrict__ n_packed, int32_t *__restrict__ unpack_index,
    int32_t *__restrict__ parent, int32_t *__restrict__ position_ids,
    uint8_t *__restrict__ tree_mask, uint64_t *__restrict__ tree_mask_bits)
{
    __shared__ int32_t s_beam[RD_MAX_N];
    __shared__ int32_t s_owner[RD_MAX_N];          // prefix_tree of this sequence
    __shared__ int32_t s_slot[RD_MAX_N];           // unpack_index of this sequence
    __shared__ int32_t s_base[RD_MAX_W + 1], s_first[RD_MAX_W + 1];
    __shared__ uint64_t s_bits[RD_MAX_N][kMaskWords];   // mask row of each packed slot
    __shared__ int s_P;

    // The dense mask, N bytes per row, is too much for one compute unit: further workgroups of the sequence repeat the
    // phases and write kMaskRows rows of it each.
    const int b = blockIdx.x, slice = blockIdx.y;
    const bool main_wg = slice == 0;
    const int tid = threadIdx.x, threads = blockDim.x;
    const int N = W * L;
    const int words = (N + 63) >> 6;
    const size_t seq = (size_t)b * N;
    RD_TR(0);
    const int ctx = ctx_len ? ctx_len[b] : 0;      // fetched with the candidates, not after them

    // N <= RD_MAX_N <= kDedupThreads: thread e owns token e = (i, j) in every per-token phase.
    static_assert(RD_MAX_N <= kDedupThreads, "one thread per token");
    const int e = tid;
    const bool tok = e < N;
    const int i = tok ? e / L : 0, j = tok ? e - i * L : 0;

    // ---- A: stage -----------------------------------------------------------------------------------
    if (tok) {
        s_beam[e] = beams[seq + e];
        s_owner[e] = i;
#pragma unroll
        for (int w = 0; w < kMaskWords; ++w) s_bits[e][w] = 0;
    }
    if (tid < W) s_first[tid] = L;
    __syncthreads();
    RD_TR(1);

    // ---- B: common prefixes of all pairs ----------------------------------------------------------------
    // Both rows are read eight tokens at a time (independent LDS reads), the match length follows
    // in registers, and the atomics that lower the owners are issued without waiting on each other.
    for (int pr = tid; pr < W * W; pr += threads) {
        const int pi = pr / W, pk = pr - pi * W;
        if (pk < pi) {
            const int32_t *ri = s_beam + pi * L, *rk = s_beam + pk * L;
            for (int j0 = 0; j0 < L; j0 += 8) {
                int32_t a[8], c[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int jj = min(j0 + t, L - 1);
                    a[t] = ri[jj];
                    c[t] = rk[jj];
                }
                int m = 0;                          // matching tokens at the head of this group
                bool run = true;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    run = run && (j0 + t < L) && (a[t] == c[t]);
                    m += run ? 1 : 0;
                }
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (t < m) atomicMin(&s_owner[pi * L + j0 + t], pk);
                if (m < 8) break;
            }
        }
    }
    rd_lds_barrier();
    RD_TR(2);

    // ---- C: first kept position per row (kept tokens are a suffix of their row) ---------------------------
    const int owner = tok ? s_owner[e] : 0;        // prefix_tree[i][j]
    if (tok && owner == i) atomicMin(&s_first[i], j);
    rd_lds_barrier();
    // exclusive prefix sum of the kept counts = first packed slot of each row (row-major slot order)
    if (tid <= W) {                                 // thread W computes the total
        int base = 0;
        for (int k = 0; k < tid; ++k) base += L - s_first[k];
        if (tid < W) s_base[tid] = base;
        else {
            s_P = base;
            if (main_wg) n_packed[b] = base;
        }
    }
    rd_lds_barrier();
    RD_TR(3);

    // ---- D: one thread per token: slot of its owner's copy -> unpack_index -----------------------------------
    if (tok) {
        const int slot = s_base[owner] + j - s_first[owner];   // (owner, j) is a kept token: j >= first_kept[owner]
        s_slot[e] = slot;
        if (main_wg) {
            unpack_index[seq + e] = slot;
            if (prefix_tree) prefix_tree[seq + e] = owner;
        }
    }
    rd_lds_barrier();

    // ---- E: one thread per kept token ---------------------------------------------------------------------------
    if (tok && owner == i) {
        const int slot = s_slot[e];
        if (main_wg) {
            packed_tokens[seq + slot] = s_beam[e];
            parent[seq + slot] = j ? s_slot[e - 1] : -1;
            position_ids[seq + slot] = ctx + j;
        }
        uint64_t path[kMaskWords];             // slots on the path from the root to (i, j)
#pragma unroll
        for (int w = 0; w < kMaskWords; ++w) path[w] = 0;
        for (int t = 0; t <= j; ++t) {
            const int q = s_slot[i * L + t];
#pragma unroll
            for (int w = 0; w < kMaskWords; ++w)
                if ((q >> 6) == w) path[w] |= 1ull << (q & 63);
        }
#pragma unroll
        for (int w = 0; w < kMaskWords; ++w) s_bits[slot][w] = path[w];
    }
    rd_lds_barrier();
    RD_TR(4);

    // ---- F: paddings and masks ---------------------------------------------------------------------------------
    const int P = s_P;
    for (int p = P + tid; p < N && main_wg; p += threads) {
        packed_tokens[seq + p] = -1;
        parent[seq + p] = -1;
        position_ids[seq + p] = -1;
    }
    if (main_wg && tree_mask_bits) {
        uint64_t *dst = tree_mask_bits + seq * words;
        for (int i = tid; i < N * words; i += threads) dst[i] = s_bits[i / words][i % words];
    }
    if (tree_mask) {
        uint8_t *dst = tree_mask + seq * N;
        const int p0 = slice * kMaskRows, rows = min(kMaskRows, N - p0);
        if ((N & 3) == 0) {                          // N*N and seq*N are multiples of 4: 32-bit stores
            uint32_t *dst4 = reinterpret_cast<uint32_t *>(dst);
            const int n4 = N >> 2;
            for (int i = tid; i < rows * n4; i += threads) {
                const int p = p0 + i / n4, q0 = (i % n4) << 2;
                const uint64_t w = s_bits[p][q0 >> 6] >> (q0 & 63);
                dst4[p * n4 + (q0 >> 2)] = (uint32_t)(w & 1) | (uint32_t)((w >> 1) & 1) << 8 |
                                           (uint32_t)((w >> 2) & 1) << 16 | (uint32_t)((w >> 3) & 1) << 24;
            }
        } else {
            for (int i = tid; i < rows * N; i += threads) {
                const int p = p0 + i / N, q = i % N;
                dst[p * N + q] = (uint8_t)((s_bits[p][q >> 6] >> (q & 63)) & 1);
            }
        }
    }
    RD_TR(5);
}

// Up to 64 tokens: a wave holds a token per lane and sets of tokens are ballots, so that nothing waits at a barrier.  All four
// waves do the same, each writes its part of the results.  Beside the launch and one round trip to memory it is bound by the
// number of its instructions (1.7 ns each in a lone wave).  us per launch in a graph, by the phases above / so: N = 16
// 3.70 / 2.05, 40 4.0 / 2.6 (without the dense mask 3.8 / 2.3), 24 sequences of 25 4.2 / 2.65; an empty launch takes 1.9.
__global__ __launch_bounds__(256) void rd_dedup_wave_kernel(
    const int32_t *__restrict__ beams, const int32_t *__restrict__ ctx_len, int W, int L, uint32_t inv_l, uint32_t inv_n,
    int32_t *__restrict__ prefix_tree, int32_t *__restrict__ packed_tokens,
    int32_t *__restrict__ n_packed, int32_t *__restrict__ unpack_index,
    int32_t *__restrict__ parent, int32_t *__restrict__ position_ids,
    uint8_t *__restrict__ tree_mask, uint64_t *__restrict__ tree_mask_bits)
{
    const int b = blockIdx.x, e = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), N = W * L;
    const size_t seq = (size_t)b * N;
    const bool tok = e < N;
    const int token = beams[seq + min(e, N - 1)];
    const int ctx = ctx_len ? ctx_len[b] : 0;
    const int i = (int)((uint32_t)e * inv_l >> 20), j = e - i * L;      // e = (candidate, position)
    auto from = [](int lane, int x) __attribute__((always_inline)) { return __builtin_amdgcn_ds_bpermute(lane * 4, x); };
    auto from64 = [&](int lane, uint64_t x) __attribute__((always_inline)) { return (uint64_t)(uint32_t)from(lane, (int)(uint32_t)x) | (uint64_t)(uint32_t)from(lane, (int)(x >> 32)) << 32; };

    // owner: the smallest candidate whose first j + 1 tokens are this one's, i.e. prefix_tree
    const uint64_t mine = ((2ull << j) - 1) << (i * L & 63);            // tokens 0 .. j of this candidate
    int owner = i;
#pragma unroll 4
    for (int k = W - 1; k >= 0; --k) {
        const uint64_t same = __ballot(token == from(k * L + j, token));
        owner = k < i && (same & mine) == mine ? k : owner;
    }
    const uint64_t kept = __ballot(tok && owner == i);                  // in the order of their slots
    const int P = __popcll(kept), slot = __popcll(kept & ((1ull << (owner * L + j)) - 1));
    if (wave == 0) {
        if (tok) {
            unpack_index[seq + e] = slot;
            if (prefix_tree) prefix_tree[seq + e] = owner;
        }
        if (e == 0) n_packed[b] = P;
    }
    // What belongs to a slot goes to the lane of that number; copies, and lanes without a token, to the first lane without a slot.
    const int to = tok && owner == i ? slot : P, before = from(e - 1, slot);
    auto place = [&](int x) __attribute__((always_inline)) { return __builtin_amdgcn_ds_permute(to * 4, x); };
    if (wave == 1) {
        const int t = place(token), up = place(j ? before : -1), pos = place(ctx + j);
        if (tok) {
            packed_tokens[seq + e] = e < P ? t : -1;
            parent[seq + e] = e < P ? up : -1;
            position_ids[seq + e] = e < P ? pos : -1;
        }
    }
    if (tree_mask == nullptr && (wave != 2 || tree_mask_bits == nullptr)) return;
    uint64_t path = 1ull << slot;                                       // slots from the root to (i, j)
    for (int d = 1; d < L; d <<= 1) {
        const uint64_t up = from64(e - d, path);
        path |= j >= d ? up : 0;
    }
    uint64_t row = (uint64_t)(uint32_t)place((int)(uint32_t)path) | (uint64_t)(uint32_t)place((int)(path >> 32)) << 32;
    row = e < P ? row : 0;                                              // of slot e
    if (wave == 2 && tok && tree_mask_bits) tree_mask_bits[seq + e] = row;
    if (tree_mask == nullptr) return;
    uint8_t *dst = tree_mask + seq * N;
    if ((N & 3) == 0) {                                                 // N*N and seq*N are multiples of 4: 32-bit stores
        const int n4 = N >> 2, all = N * n4;
        for (int t0 = wave * 64; t0 < all; t0 += 256) {
            const int t = t0 + e, p = (int)((uint32_t)t * inv_n >> 20), q = t - p * n4;
            const uint32_t w = (uint32_t)(from64(p, row) >> (q * 4 & 63)) & 15u;
            if (t < all) reinterpret_cast<uint32_t *>(dst)[t] = (w * 0x00204081u) & 0x01010101u;      // a bit to a byte
        }
    } else {
        for (int t0 = wave * 64; t0 < N * N; t0 += 256) {
            const int t = t0 + e, p = (int)((uint32_t)t * inv_n >> 20), q = t - p * N;
            const uint64_t w = from64(p, row) >> (q & 63);
            if (t < N * N) dst[t] = (uint8_t)(w & 1);
        }
    }
}

// More than 64 tokens, up to 64 to a candidate: a token per lane, whole candidates per wave (64 / L of them), and sets of a wave's
// tokens are ballots.  A wave compares its candidates with every one before them, whose tokens all lanes of a position read from
// one place in LDS (unrolled, so that the reads run ahead); three barriers in all.  Bound by that loop, some 45 clocks a candidate,
// beside the launch and one round trip to memory.  The phases of rd_dedup_kernel, with the pairs of candidates shared out to 1024
// threads and the owners lowered by atomics, took longer, above all for the serial sums over candidates and positions.  us per launch
// in a graph, those phases / this: N = 80 3.8 / 3.2, 16 sequences of it with the dense mask 4.5 / 3.85, N = 150 4.7 / 4.1, 350 8.9 / 6.8,
// with the mask 11.1 / 7.6, 24 sequences of it 16.7 / 8.85; 128 candidates of 3 tokens 18.0 / 9.7; 2 of 64 11.5 / 6.0.  (Prefixes
// compared by 32-bit halves, without the order of candidates outside the wave: 350 7.65.)
__global__ __launch_bounds__(kMaxTokenWaves * 64) void rd_dedup_waves_kernel(
    const int32_t *__restrict__ beams, const int32_t *__restrict__ ctx_len, int W, int L, int per_wave, int token_waves, uint32_t inv_l, uint32_t inv_w, uint32_t inv_n4, uint32_t inv_n2,
    int32_t *__restrict__ prefix_tree, int32_t *__restrict__ packed_tokens,
    int32_t *__restrict__ n_packed, int32_t *__restrict__ unpack_index,
    int32_t *__restrict__ parent, int32_t *__restrict__ position_ids,
    uint8_t *__restrict__ tree_mask, uint64_t *__restrict__ tree_mask_bits)
{
    __shared__ int32_t s_beam[RD_MAX_N];
    __shared__ __align__(8) uint32_t s_bits[RD_MAX_N * kMaskWords * 2];      // mask row of each packed slot
    __shared__ uint64_t s_kept[kMaxTokenWaves];
    const int b = blockIdx.x, slice = blockIdx.y;
    const bool main_wg = slice == 0;               // (further ones: rows of the dense mask, as in rd_dedup_kernel)
    const int tid = threadIdx.x, threads = blockDim.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = W * L, words = (N + 63) >> 6;
    const size_t seq = (size_t)b * N;
    const int own = (int)((uint32_t)lane * inv_l >> 20), j = lane - own * L;      // candidate in the wave, position
    const int i = wave * per_wave + own, e = i * L + j;
    const bool tok = own < per_wave && i < W;
    const int token = beams[seq + min(e, N - 1)];
    const int ctx = ctx_len ? ctx_len[b] : 0;
    if (tok) s_beam[e] = token;
    for (int t = tid; t < N * words * 2; t += threads) s_bits[t] = 0;
    rd_lds_barrier();

    // owner: the smallest candidate whose first j + 1 tokens are this one's, i.e. prefix_tree
    const uint64_t mine = ((2ull << j) - 1) << (own * L & 63);          // tokens 0 .. j of this candidate
    int owner = i;
    if (wave < token_waves) {
#pragma unroll 8
        for (int k = min((wave + 1) * per_wave, W) - 2; k >= 0; --k) {
            const uint64_t same = __ballot(token == s_beam[k * L + j]);
            owner = k < i && (same & mine) == mine ? k : owner;
        }
        const uint64_t kept = __ballot(tok && owner == i);              // in the order of their slots
        if (lane == 0) s_kept[wave] = kept;
    }
    rd_lds_barrier();
    const int there = (int)((uint32_t)owner * inv_w >> 20);             // the owner's wave
    int slot = __popcll(s_kept[tok ? there : 0] & ((1ull << (((owner - there * per_wave) * L + j) & 63)) - 1)), P = 0;
    for (int w = 0; w < token_waves; ++w) {
        const int n = __popcll(s_kept[w]);
        slot += w < there ? n : 0;
        P += n;
    }
    const bool keep = tok && owner == i;          // (waves beyond the tokens only help to write)
    const int up = __builtin_amdgcn_ds_bpermute((lane - 1) * 4, slot);
    if (main_wg) {
        if (tid == 0) n_packed[b] = P;
        if (tok) {
            unpack_index[seq + e] = slot;
            if (prefix_tree) prefix_tree[seq + e] = owner;
        }
        if (keep) {
            packed_tokens[seq + slot] = token;
            parent[seq + slot] = j ? up : -1;
            position_ids[seq + slot] = ctx + j;
        }
        for (int p = P + tid; p < N; p += threads) packed_tokens[seq + p] = parent[seq + p] = position_ids[seq + p] = -1;
    }
    // the slots from the root to (i, j)
    for (int t = 0; t < L; ++t) {
        const int q = __builtin_amdgcn_ds_bpermute((own * L + t) * 4, slot);
        if (keep && t <= j) atomicOr(&s_bits[slot * words * 2 + (q >> 5)], 1u << (q & 31));
    }
    rd_lds_barrier();
    if (main_wg && tree_mask_bits) {
        uint64_t *dst = tree_mask_bits + seq * words;
        for (int t = tid; t < N * words; t += threads) dst[t] = reinterpret_cast<const uint64_t *>(s_bits)[t];
    }
    if (tree_mask) {
        uint8_t *dst = tree_mask + seq * N;
        const int p0 = slice * kMaskRows, rows = min(kMaskRows, N - p0);
        if ((N & 3) == 0) {                          // N*N and seq*N are multiples of 4: 32-bit stores
            uint32_t *dst4 = reinterpret_cast<uint32_t *>(dst);
            const int n4 = N >> 2;
            for (int t = tid; t < rows * n4; t += threads) {
                const int r = (int)((uint32_t)t * inv_n4 >> 20), p = p0 + r, q = (t - r * n4) * 4;
                const uint32_t w = s_bits[p * words * 2 + (q >> 5)] >> (q & 31) & 15u;
                dst4[p * n4 + (q >> 2)] = (w * 0x00204081u) & 0x01010101u;      // a bit to a byte
            }
        } else if ((N & 1) == 0) {                   // the same, by pairs, which lie in one row each: N*N is a multiple of 4, the rows are even in number
            uint32_t *dst4 = reinterpret_cast<uint32_t *>(dst + p0 * N);
            const int n2 = N >> 1, pairs = rows * n2;
            auto pair = [&](int t) __attribute__((always_inline)) {
                const int r = (int)((uint64_t)(uint32_t)t * inv_n2 >> 24), p = p0 + r, q = (t - r * n2) * 2;
                return s_bits[p * words * 2 + (q >> 5)] >> (q & 31) & 3u;
            };
            for (int t = tid * 2; t < pairs; t += threads * 2) dst4[t >> 1] = (pair(t) * 0x81u & 0x101u) | (pair(t + 1) * 0x810000u & 0x1010000u);
        } else {
            for (int t = tid; t < rows * N; t += threads) {
                const int p = p0 + t / N, q = t % N;
                dst[p * N + q] = (uint8_t)(s_bits[p * words * 2 + (q >> 5)] >> (q & 31) & 1);
            }
        }
    }
}

}  // namespace

extern "C" int rd_dedup(const int32_t *beams, const int32_t *ctx_len, int B, int W, int L,
                        int32_t *prefix_tree, int32_t *packed_tokens, int32_t *n_packed,
                        int32_t *unpack_index, int32_t *parent, int32_t *position_ids,
                        uint8_t *tree_mask, uint64_t *tree_mask_bits, void *stream)
{
    const int st = rd_check_beam_shape(B, W, L);
    if (st != RD_OK) return st;
    if (!beams || !packed_tokens || !n_packed || !unpack_index || !parent || !position_ids)
        return RD_ERR_INVALID_ARG;
    if (!rd_aligned(tree_mask, 4) || !rd_aligned(tree_mask_bits, 8)) return RD_ERR_INVALID_ARG;
    const int N = W * L;
    if (N <= 64) {
        // x / d = x * inv >> 20 for x below 4096 and d up to 64 (x * (d - 1) < 2^20)
        auto inverse = [](int d) { return ((1u << 20) + (uint32_t)d - 1) / (uint32_t)d; };
        hipLaunchKernelGGL(rd_dedup_wave_kernel, dim3(B), dim3(256), 0, (hipStream_t)stream, beams, ctx_len, W, L, inverse(L),
                           inverse((N & 3) == 0 ? N >> 2 : N), prefix_tree, packed_tokens, n_packed, unpack_index, parent, position_ids,
                           tree_mask, tree_mask_bits);
        return rd_check_launch();
    }
    const int slices = tree_mask ? (W * L + kMaskRows - 1) / kMaskRows : 1;
    if (L <= 64) {
        // as above; candidates below 128 by up to 32 in a wave, words of kMaskRows rows by up to 96
        auto inverse = [](int d) { return ((1u << 20) + (uint32_t)d - 1) / (uint32_t)d; };
        const int per_wave = 64 / L, waves = (W + per_wave - 1) / per_wave;
        hipLaunchKernelGGL(rd_dedup_waves_kernel, dim3(B, slices), dim3((tree_mask && waves < kMaskWaves ? kMaskWaves : waves) * 64), 0,
                           (hipStream_t)stream, beams, ctx_len, W, L, per_wave, waves, inverse(L), inverse(per_wave), inverse(N >> 2),
                           ((1u << 24) + (uint32_t)(N >> 1) - 1) / (uint32_t)(N >> 1), prefix_tree, packed_tokens, n_packed, unpack_index, parent,
                           position_ids, tree_mask, tree_mask_bits);
        return rd_check_launch();
    }
    hipLaunchKernelGGL(rd_dedup_kernel, dim3(B, slices), dim3(kDedupThreads), 0, (hipStream_t)stream,
                       beams, ctx_len, W, L, prefix_tree, packed_tokens, n_packed, unpack_index,
                       parent, position_ids, tree_mask, tree_mask_bits);
    return rd_check_launch();
}
