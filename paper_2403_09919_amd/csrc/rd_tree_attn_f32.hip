// rd_tree_attn, fp32: for fp32 Q/K/V, where results must hold to ~1e-6, on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, twice the rate of the vector units).
//
// The keys of a head are a sequence of 16-key tiles, the context's first, then the packed keys'; wave w of a workgroup
// takes tiles w, w + 8, ... and keeps a softmax state of its own.  Nothing but Q passes through LDS in the loop:
//   * S^T = K Q^T: the A operand is K as loaded, lane (r16, g) = key r16, floats 16c + 4g .. +3 (the order of the
//     contraction is free as long as Q's is the same);
//   * O^T = V^T P^T: a lane's four scores are keys 4g+i of row r16; step i of the product takes exactly those, so the
//     probabilities are the B operand as they are, and the A operand is V as loaded, lane (r16, g) = floats
//     64jj + 4 r16 .. +3 of key 4g+i (d-tile e of jj holds d = 64jj + 4m + e).
// The next tile's K and V are in flight meanwhile; the eight states meet in LDS once, at the end.
// Short contexts are bound by latency, long ones by the block's chain of loads and products (3 us per 128 keys and
// workgroup at D = 128), wide beams by the matrix unit.  One row tile per workgroup: two share a tile's loads but
// lengthen every chain (7.6 against 5.5 us at the first shape below, 117 against 136 us at the last but one), and K/V of a
// head's row groups come from L2.  Against vector arithmetic on LDS tiles with the packed keys as a workgroup of their
// own, us per launch: H=4, C=128, D=64, 9 packed rows 14.4 -> 5.15; B=3, H=26, C=250 56.7 -> 13.6; H=10, C=3000 43 -> 16.5;
// H=5, C=1000, 52 rows 64.7 -> 13.4; B=4, H=40, C=2000, 33 rows 453 -> 117; B=8, H=32, C=1500 487 -> 101.
#include "rd_attn_common.h"
#include <type_traits>

namespace rd {

constexpr int kF32Waves = 8;

// A workgroup takes one row tile (16 packed rows); more rows are row groups.
template <int D>
__global__ __launch_bounds__(kF32Waves * 64, 2) void rd_tree_attn_f32_kernel(AttnArgs a)
{
    constexpr int NW = kF32Waves;
    constexpr int KC = D / 16;                                  // 16-byte pieces of a row per lane group
    constexpr int JJ = D / 64;                                  // 64-column pieces of the output
    constexpr int kRows = 16;
    constexpr int kUnits = JJ * 4;                              // output fragments: (jj, i), 64 lanes x 4 floats
    static_assert(kUnits <= NW && KC <= NW, "a wave finishes one output fragment and brings in one of Q");
    constexpr int kPF = kRows * 2 + kUnits * 256;               // floats per partial: (m,l) per row, then the fragments
    constexpr int kMLStride = NW * 2 + 4;                       // floats per row of the waves' (m, l) table
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    f32x4 *sQ = reinterpret_cast<f32x4 *>(smem);                // [KC][64 lanes]
    f32x4 *sO = sQ + KC * 64;                                   // [NW][kUnits][64 lanes]
    float *sML = reinterpret_cast<float *>(sO + NW * kUnits * 64);   // [kRows][NW] (m, l)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;

    // which (sequence, head) -- all workgroups of one on one XCD (10 heads, C=3000: 18.7 us, spread over all 19.4; 5 heads,
    // C=6000: 19.9 and 20.7) -- and which of its a.S workgroups
    const int k = (int)(blockIdx.x >> 3);
    const int hl = a.S == 1 ? k : k / a.S;
    const int r_wg = k - hl * a.S;
    const int bh = hl * 8 + (int)(blockIdx.x & 7);
    if (bh >= a.B * a.H) return;
    const int b = a.B == 1 ? 0 : bh / a.H;
    const int C = clampi(a.ctx_len[b], 0, a.Cmax);
    const int P_all = clampi(a.n_packed[b], 0, a.N);
    // row groups with packed rows share the head's workgroups; output rows of the others are zero
    const int n_act = a.n_rg == 1 ? 1 : max((P_all + kRows - 1) / kRows, 1);
    const int ranges = n_act == 1 ? a.S : a.S / n_act;
    const int split = n_act == 1 ? r_wg : r_wg / n_act;
    const int rg = r_wg - split * n_act;
    if (a.n_rg > 1) {
        float *z = static_cast<float *>(a.out) + (size_t)bh * a.N * D;
        for (int i = n_act * kRows * D + (r_wg * NW * 64 + tid) * 4; i < a.N * D; i += a.S * NW * 64 * 4)
            *reinterpret_cast<float4 *>(z + i) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (split >= ranges) return;
    const int row0 = rg * kRows;
    const int P = clampi(P_all - row0, 0, kRows);
    const int Ng = min(kRows, a.N - row0);
    const int tree_end = min(P_all, row0 + kRows);              // (the mask is lower triangular)

    const int nA = (C + 15) >> 4;
    const int nT = P > 0 ? nA + ((tree_end + 15) >> 4) : 0;
    const int nblk = (nT + NW - 1) / NW;
    const int per = ranges == 1 ? max(nblk, 1) : max((nblk + ranges - 1) / ranges, 1);
    const int n_part = ranges == 1 ? 1 : max((nblk + per - 1) / per, 1);
    if (split >= n_part) return;
    const int tile_begin = split * per * NW;
    const int tile_end = min(nT, tile_begin + per * NW);

    const float *Qb = static_cast<const float *>(a.q) + ((size_t)bh * a.N + row0) * D;
    const uintptr_t Kc = reinterpret_cast<uintptr_t>(a.k_cache) + (size_t)bh * a.Cmax * D * 4;
    const uintptr_t Vc = reinterpret_cast<uintptr_t>(a.v_cache) + (size_t)bh * a.Cmax * D * 4;
    const uintptr_t Kn = reinterpret_cast<uintptr_t>(a.k_new) + (size_t)bh * a.N * D * 4 - Kc;   // from the cache's rows to the packed ones
    const uintptr_t Vn = reinterpret_cast<uintptr_t>(a.v_new) + (size_t)bh * a.N * D * 4 - Vc;
    typedef const __attribute__((address_space(1))) f32x4 gvec;

    // Q is asked for before K and V: loads return in order, and a wave that asks for it last, as the compiler would by the use
    // below, meets the others at the barrier only when all of its first tile has come.  us by Q last / Q first: H=8, D=128,
    // C=55 7.60 / 6.67; B=53, H=40, C=147, 24 x 4 tokens 569 / 490; B=7, H=52, C=214 30.7 / 28.7; D=64, B=6, H=32, C=101 5.27 /
    // 4.91; B=11, H=52, C=200 21.4 / 21.0; over 200 launches of 17 to 4400 keys 5 % less in the mean, none longer.
    // (The first two tiles of a wave asked for together, without a loop: as fast where the second is not there, slower
    // where it is: 32.8 and 23.7 us at the third and the last of these.)
    f32x4 qreg;
    const bool q_wave = KC >= NW || wave < KC;
    if (q_wave) qreg = *reinterpret_cast<const f32x4 *>(Qb + (size_t)min(r16, Ng - 1) * D + wave * 16 + g * 4);
    __builtin_amdgcn_sched_barrier(0);

    // K, V and visibility words of a tile.  A wave whose turn falls past the end takes the last tile again (masked), a
    // workgroup without tiles the first there is: no branch around the loads.  Rows past a tile's keys are its last key.
    f32x4 kreg[KC], vreg[4][JJ];
    uint64_t mword;
    auto fetch = [&](int tile, auto which_k, auto which_v) __attribute__((always_inline)) {
        const int tl = max(min(tile, tile_end - 1), 0);
        const bool tree = tl >= nA;
        const int first = (tl - (tree ? nA : 0)) * 16;
        const int keys = max(min(16, (tree ? tree_end : C) - first), 1);
        if (decltype(which_k)::value) {
            const uintptr_t p = Kc + (tree ? Kn : 0) + (size_t)first * D * 4 + (uint32_t)min(r16, keys - 1) * (D * 4) + g * 16;
#pragma unroll
            for (int c = 0; c < KC; ++c) kreg[c] = *(gvec *)(p + c * 64);
            const int word = tree ? min(first >> 6, a.words - 1) : 0;
            mword = a.mask_bits[((size_t)b * a.N + min(row0 + r16, a.N - 1)) * a.words + word];
        }
        if (decltype(which_v)::value) {
            const uintptr_t p = Vc + (tree ? Vn : 0) + (size_t)first * D * 4 + r16 * 16;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int jj = 0; jj < JJ; ++jj) vreg[i][jj] = *(gvec *)(p + (uint32_t)min(4 * g + i, keys - 1) * (D * 4) + jj * 256);
        }
    };
    using yes = std::true_type;
    using no = std::false_type;
    const int t_first = tile_begin + wave;
    fetch(t_first, yes{}, yes{});

    if (q_wave) sQ[wave * 64 + lane] = r16 < P ? qreg : f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 oacc[JJ][4];
#pragma unroll
    for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[jj][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    rd_lds_barrier();         // Q visible to all waves

    auto tile_step = [&](int tile, auto more) __attribute__((always_inline)) {
        const bool tree = tile >= nA;
        const int first = (tile - (tree ? nA : 0)) * 16;
        const int rem = (tree ? tree_end : C) - first;          // keys of the tile inside the range
        const uint32_t vis = tree ? (uint32_t)(mword >> ((first & 63) + 4 * g)) & 0xfu : 0xfu;
        const int left = rem - 4 * g;
        const uint32_t tail = left >= 4 ? 0xfu : (left <= 0 ? 0u : (1u << left) - 1u);
        const uint32_t bits = r16 < P ? vis & tail : 0u;
        f32x4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const f32x4 q = sQ[c * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_16x16x4f32(kreg[c][e], q[e], sacc, 0, 0, 0);
        }
        if (decltype(more)::value) fetch(tile + NW, yes{}, no{});
        float s[4], p[4], mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = (bits >> i) & 1u ? sacc[i] * a.scale_log2e : -INFINITY;
            mx = fmaxf(mx, s[i]);
        }
        const float m_new = fmaxf(m_run, quad_max(mx));
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        m_run = m_new;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f(s[i] - m_safe);
            sum += p[i];
        }
        l_run = l_run * alpha + sum;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[jj][e] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[jj][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vreg[i][jj][e], p[i], oacc[jj][e], 0, 0, 0);
        if (decltype(more)::value) fetch(tile + NW, no{}, yes{});
    };
    if (t_first < tile_end) {
        int tile = t_first;
        for (; tile + NW < tile_end; tile += NW) tile_step(tile, yes{});
        tile_step(tile, no{});
    }

    // ---- the waves' states meet in LDS; fragment (jj, i) holds, per lane, d = 64jj + 16g + 4i .. +3 of row r16
    const float l_sum = quad_sum(l_run);
    if (g == 0) *reinterpret_cast<float2 *>(sML + r16 * kMLStride + wave * 2) = make_float2(m_run, l_sum);
#pragma unroll
    for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            sO[(wave * kUnits + jj * 4 + i) * 64 + lane] = f32x4{oacc[jj][0][i], oacc[jj][1][i], oacc[jj][2][i], oacc[jj][3][i]};
    rd_lds_barrier();
    const int n_waves = clampi(tile_end - tile_begin, 1, NW);   // waves that had a tile
    const int f = min(wave, kUnits - 1);                        // this wave's fragment of the output
    f32x4 ml[NW / 2];
#pragma unroll
    for (int w = 0; w < NW / 2; ++w) ml[w] = *reinterpret_cast<const f32x4 *>(sML + r16 * kMLStride + w * 4);
    float fm = -INFINITY, fl = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) fm = fmaxf(fm, ml[w / 2][2 * (w & 1)]);
    const float ms = fm == -INFINITY ? 0.f : fm;
    f32x4 fo = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](int w) __attribute__((always_inline)) {
        const float s = __builtin_amdgcn_exp2f(ml[w / 2][2 * (w & 1)] - ms);
        fl += s * ml[w / 2][2 * (w & 1) + 1];
        fo += s * sO[(w * kUnits + f) * 64 + lane];
    };
#pragma unroll
    for (int w = 0; w < NW / 2; ++w) add(w);
    if (n_waves > NW / 2) {
#pragma unroll
        for (int w = NW / 2; w < NW; ++w) add(w);
    }

    float *outp = static_cast<float *>(a.out) + ((size_t)bh * a.N + row0) * D;
    auto put = [&](f32x4 o, float l) __attribute__((always_inline)) {
        if (wave < kUnits && r16 < Ng) {
            const float inv = r16 < P ? 1.0f / l : 0.f;         // rows beyond the packed count are zero
            f32x4 y = o * inv;
            if (r16 >= P) y = f32x4{0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4 *>(outp + (size_t)r16 * D + (f / 4) * 64 + g * 16 + (f & 3) * 4) = y;
        }
    };
    if (n_part == 1) {
        put(fo, fl);
        return;
    }
    // ---- partial state -> workspace; the last workgroup of this head (and row group) merges
    const size_t unit = (size_t)bh * a.n_rg + rg;
    float *part = a.partials + ((size_t)bh * a.S + split * n_act + rg) * kPF;
    const bool real = wave < kUnits && r16 < P;
    if (real) {
        if (f == 0 && g == 0) st_dev2(part + 2 * r16, fm, fl);
        st_dev4(part + 2 * kRows + f * 256 + lane * 4, fo[0], fo[1], fo[2], fo[3]);
    }
    const int last = arrive_is_last(a.counters + unit, (uint32_t)n_part);
    if (last == kNotLast) return;
    const bool cached = last == kLastClean;
    constexpr int kChunk = 8;                                   // partials whose loads are in flight together
    const float *hp = a.partials + ((size_t)bh * a.S + rg) * kPF;
    float M = -INFINITY, den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s0 = 0; s0 < n_part; s0 += kChunk) {
        float2 pml[kChunk];
        f32x4 pfr[kChunk];
#pragma unroll
        for (int c = 0; c < kChunk; ++c) {
            pml[c] = make_float2(-INFINITY, 0.f);               // absent: weight 2^-inf = 0
            pfr[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (s0 + c < n_part && real) {
                const float *ps = hp + (size_t)(s0 + c) * n_act * kPF, *pf = ps + 2 * kRows + f * 256 + lane * 4;
                if (cached) {
                    pml[c] = *reinterpret_cast<const float2 *>(ps + 2 * r16);
                    pfr[c] = *reinterpret_cast<const f32x4 *>(pf);
                } else {
                    pml[c] = ld_dev2(ps + 2 * r16);
                    const float2 lo = ld_dev2(pf), hi = ld_dev2(pf + 2);
                    pfr[c] = f32x4{lo.x, lo.y, hi.x, hi.y};
                }
            }
        }
        float Mn = M;
#pragma unroll
        for (int c = 0; c < kChunk; ++c) Mn = fmaxf(Mn, pml[c].x);
        const float Ms = Mn == -INFINITY ? 0.f : Mn, resc = __builtin_amdgcn_exp2f(M - Ms);
        den *= resc;
        acc *= resc;
#pragma unroll
        for (int c = 0; c < kChunk; ++c) {
            const float w = __builtin_amdgcn_exp2f(pml[c].x - Ms);
            den += w * pml[c].y;
            acc += w * pfr[c];
        }
        M = Mn;
    }
    put(acc, den);
    if (tid == 0) a.counters[unit] = 0;       // leave the workspace ready for the next call
}

template <int D>
static int launch_f32(const AttnArgs &a, hipStream_t stream)
{
    constexpr size_t smem = (size_t)(D / 16) * 1024 + (size_t)kF32Waves * (D / 16) * 1024 + (size_t)16 * (kF32Waves * 2 + 4) * sizeof(float);
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    static std::atomic<unsigned long long> configured{0};
    const int st = ensure_dynamic_lds(reinterpret_cast<const void *>(&rd_tree_attn_f32_kernel<D>), smem, configured);
    if (st != RD_OK) return st;
    const size_t wgs = ((size_t)a.B * a.H + 7) / 8 * 8 * a.S;
    if (wgs > 0x7fffffffull) return RD_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((rd_tree_attn_f32_kernel<D>), dim3((unsigned)wgs), dim3(kF32Waves * 64), smem, stream, a);
    return rd_check_launch();
}

int tree_attn_f32(const AttnArgs &a, int D, hipStream_t stream)
{
    return D == 128 ? launch_f32<128>(a, stream) : launch_f32<64>(a, stream);
}

}  // namespace rd
