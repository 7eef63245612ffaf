// Tree-masked attention of the packed candidates against the KV cache (Sec. 3.3, 3.4) on the gfx950 matrix cores
// for 16-bit K/V (bf16 or fp16): a split-key flash kernel, its template and dispatch, instantiated per element
// type, cache layout and rotation (rd_tree_attn_bf16.hip, _f16, _paged, _rope_bf16, _rope_f16).
//
// A key range is a sequence of 32-key tiles, the context's first, then the packed keys'; a block is NW of them, one
// per wave.  Per block a wave
//   * has K of its tile in registers as the A operand of S^T = K Q^T and Q there too as the B operand;
//   * takes the softmax of its 32 keys and leaves the probabilities in LDS as its lanes hold them (keys of a tile
//     taken as 4g+i, 16+4g+i: that is the B-operand order of the next product), beside its V tile;
//   * after one barrier adds up its own d-tiles of O^T = V^T P^T over all the block's tiles; V^T (eight keys of one
//     column per lane) comes from the row-major V tiles by transpose reads.
// The next block's K and V are in flight meanwhile.
//
// What bounds it.  Long contexts in large batches: HBM (43.5 us for 201 MB of K and V at B=8, H=32, C=1536, 4.6 TB/s).
// Everything else: latency -- loads in operand order (see stage_k), and per block the LDS traffic, the vector
// arithmetic of the softmax and the matrix products, which two waves per SIMD in step overlap badly.  Hence: one
// barrier where the data is ready and one where it is free, no exchange of maxima in between (kSlack); tiles of the
// context and of the tree in one sequence, so that a short context and its tree are one block and one workgroup;
// no more workgroups per head than the lengths at hand need (n_part).  Against the kernel it replaced, whose waves
// met at three barriers per block and whose packed keys were a workgroup of their own at short contexts, us per
// launch, K and V from memory: H=8, C=87, 20 packed rows 9.3 -> 5.4; B=11, H=40, C=180 36.0 -> 16.1; B=20, H=26, C=300,
// D=64 21.4 -> 16.7; H=32, C=1024 12.7 -> 12.1; H=32, C=1777, 147 rows 33.9 -> 30.0; B=8, H=32, C=1536 45.8 -> 43.5;
// B=4, H=40, C=4096, 27 to 38 rows of 80 76.4 -> 74.4; nothing at B=6, H=40, C=700, 83 to 130 rows (53.9 -> 53.4) and
// B=16, H=52, C=2048 (182.6 -> 183.3).
#pragma once
#include "rd_attn_common.h"
#include <type_traits>

#ifdef RD_TRACE
extern __device__ unsigned long long *rd_trace_buf;     // defined by the including file (RD_TRACE_DEFINE)
#endif

namespace rd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
// 16-bit element types of the MFMA kernels: eight-element operand vector and the matrix instruction
template <typename T> struct Elem;
template <> struct Elem<__bf16> {
    typedef bf16x8 vec8;
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Elem<_Float16> {
    typedef f16x8 vec8;
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int D>
struct Geo {
    static constexpr int kChunks = D / 8;                  // 16-byte chunks per row
    static constexpr int kRowBytes = D * 2;
    static constexpr int kTileKeys = 32;                   // keys per wave per block
    static constexpr int kRowsPerLoad = 64 / kChunks;      // rows one wave-wide 16-byte load covers
    static constexpr int kLoads = kTileKeys / kRowsPerLoad;  // loads per wave per tile
    static constexpr int kTileBytes = kTileKeys * kRowBytes;
    static constexpr int kKSteps = D / 32;                 // MFMA k-steps of the QK^T contraction
    static constexpr int kDTiles = D / 16;
};

// LDS placement of 16-byte chunk c of row `row`: K tiles are read by 16 lanes holding 16
// different rows and one chunk index, V tiles by transpose reads that touch 8 rows x 2 adjacent
// chunks per half-wave; each gets the XOR pattern that spreads its readers over all banks.
template <int D> __device__ __forceinline__ int kswz(int row, int c) { return c ^ (row & (Geo<D>::kChunks - 1)); }
template <int D> __device__ __forceinline__ int vswz(int row, int c)
{
    return ((((c >> 1) ^ (row & (Geo<D>::kChunks / 2 - 1))) << 1) | (c & 1));
}

__device__ __forceinline__ uint4 ldg16(const void *p) { return *reinterpret_cast<const uint4 *>(p); }

// Synchronisation that orders LDS traffic only.  __syncthreads() also waits for every global
// load in flight, which would drain the K/V prefetch at each of the barriers per block.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// Orders this wave's own LDS writes before its own later LDS reads (tiles private to a wave).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Rotary embedding of eight elements ("rotate half": element i pairs with element i + D/2), in the
// arithmetic of rd_rope: fp32, the partner's product rounded, then one fused multiply-add, one rounding to
// the storage type.  `x` is this lane's 16-byte chunk, `partner` the chunk D/2 elements away in the same row,
// cs / sn the cosines and sines of the eight pairs; `low`: x is the lower half of the pairs.
template <typename T>
__device__ __forceinline__ uint4 rope8(uint4 x, uint4 partner, const float (&cs)[8], const float (&sn)[8], bool low)
{
    typedef typename Elem<T>::vec8 vec8;
    const vec8 xv = __builtin_bit_cast(vec8, x), pv = __builtin_bit_cast(vec8, partner);
    vec8 y;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float a = (float)xv[i], b = (float)pv[i];
        float ps = b * sn[i];
        asm volatile("" : "+v"(ps));              // an fp32 product, then one fused multiply-add
        float r = __builtin_fmaf(a, cs[i], low ? -ps : ps);
        asm volatile("" : "+v"(r));               // an fp32 sum, then one rounding (as rd_rope does)
        y[i] = (T)r;
    }
    return __builtin_bit_cast(uint4, y);
}

// Row tiles (16 packed rows) of a workgroup at most: what registers and LDS hold.
constexpr int kMaxTiles = 5;
constexpr int kGroupTiles = 4;      // ... where beams have more packed keys than a block holds

// Whether K is fetched as whole rows and turned into operand order through LDS (16 keys at a time, 32 KB for eight
// waves), or fetched in operand order (lane = key r16 x 16-byte chunk 4t+g).  In operand order the 16 lanes of a row
// touch 16 cache lines, which costs about 1 us per 64 KB: eight-wave workgroups, chosen where there are too few to
// fill the chip, are bound by that (17.3 against 19.0 us at H=32, C=1024 in one workgroup per head).  With two
// four-wave workgroups per compute unit the other one's work covers it (B=11, H=40, C=180: 13.1 us, 15.2 staged), and
// with five row tiles the LDS is not there.
template <int D, int NQ, int NW> constexpr bool stage_k() { return NW == 8 && NQ <= 4; }

// NW = waves per workgroup (4 or 8); NQ = row tiles; TB = packed-key tiles a wave can meet (1 for all but the widest
// beams: the mask words of all of them are fetched up front).
// PAGED: the context keys and values live in fixed-size pages found through a block table
// (a.block_table, a.page_size, a.max_pages) instead of one dense [B,H,Cmax,D] tensor.
// ROPE: q and k_new arrive unrotated; the kernel applies the rotary embedding at a.position_ids
// to the query rows as it brings them into LDS and to the packed-key tiles as it walks them.
template <typename T, int D, int NQ, int NW, int TB, bool PAGED, bool ROPE>
__global__ __launch_bounds__(NW * 64, 2) void rd_tree_attn_mfma_kernel(AttnArgs a)
{
    using G = Geo<D>;
    using vec8 = typename Elem<T>::vec8;
    constexpr int KS = G::kKSteps;
    constexpr int DT = G::kDTiles;
    constexpr int kRows = NQ * 16;
    constexpr int JW = DT >= NW ? DT / NW : 1;                  // d-tiles of the output a wave owns
    constexpr int RW = DT >= NW ? 1 : NW / DT;                  // waves that share d-tiles and divide the row tiles
    constexpr int QW = (NQ + RW - 1) / RW;                      // row tiles of a wave's output
    constexpr int kPF = kRows * 2 + DT * NQ * 256;              // floats per partial: (m,l) per row, then fragments
    constexpr bool kStageK = stage_k<D, NQ, NW>();
    constexpr bool kQReg = NQ * KS <= 8;                       // Q operands stay in registers
    constexpr int kMLStride = NW * 8 + 16;                      // bytes per row of the tiles' (maximum, sum) table
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *sQ = smem;                                   // [NQ][KS][64 lanes] x 16 B, B-operand order
    unsigned char *sV = sQ + NQ * KS * 1024;                    // [NW] V tiles
    unsigned char *sP = sV + NW * G::kTileBytes;                // [NW][NQ][64 lanes] x 16 B
    unsigned char *sML = sP + NW * NQ * 1024;                   // [kRows] x [NW] (maximum, sum)

    constexpr bool kVisInLds = NQ > 4;                          // the visibility bytes: registers, or LDS where those are short
    int *sMoved = reinterpret_cast<int *>(sML + kRows * kMLStride);             // [NW] a reference moved in the wave's tile
    unsigned char *sVis = reinterpret_cast<unsigned char *>(sMoved + NW);       // [TB][NW][NQ][64 lanes]
    unsigned char *sK = sVis;                                   // [NW] half K tiles (kernels without sVis)
    constexpr float kSlack = 8.f;                               // exponents may exceed their reference by this much

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15;
    const int g = lane >> 4;
    RD_TR(0);

    // ---- which (sequence, head), which of its a.S workgroups.  Workgroups are dealt round-robin to the 8 XCDs; all of
    // a head's go to one of them, whose L2 then serves Q, K/V shared by row groups and the partial results (merging
    // partials past the L2 takes about twice as long).  Head numbers past the end fill up the last eight.  So too with
    // fewer than eight heads, which leaves XCDs idle: spread over all of them, 30 of 31 shapes are slower (us, on one
    // XCD / spread: 1 head, C=32000 32.0 / 33.5; 4 heads, C=8000 18.7 / 20.1; 5 heads, C=16000 24.4 / 26.2; 12 heads, C=4000
    // 17.1 / 17.4; 26 heads, C=6000 27.0 / 28.1), the one being 10 heads, C=6000 and 350 tokens (38.7 / 33.1).
    const int k = (int)(blockIdx.x >> 3);
    const int hl = a.S == 1 ? k : k / a.S;
    const int r_wg = k - hl * a.S;
    const int bh = hl * 8 + (int)(blockIdx.x & 7);
    if (bh >= a.B * a.H) return;
    const int b = a.B == 1 ? 0 : bh / a.H;
    const int n_rg = a.n_rg;
    const int C = clampi(a.ctx_len[b], 0, a.Cmax);
    const int P_all = clampi(a.n_packed[b], 0, a.N);
    // Row groups that hold packed rows share the head's workgroups evenly (a.S >= n_rg); a workgroup is
    // (row group rg, key range split).  Output rows of the other groups are zero.
    const int n_act = n_rg == 1 ? 1 : max((P_all + kRows - 1) / kRows, 1);
    const int ranges = n_act == 1 ? a.S : a.S / n_act;
    const int split = n_act == 1 ? r_wg : r_wg / n_act;
    const int rg = r_wg - split * n_act;
    if (n_rg > 1) {
        T *z = static_cast<T *>(a.out) + (size_t)bh * a.N * D;
        for (int i = n_act * kRows * D + (r_wg * NW * 64 + tid) * 8; i < a.N * D; i += a.S * NW * 64 * 8)
            *reinterpret_cast<uint4 *>(z + i) = make_uint4(0, 0, 0, 0);
    }
    if (split >= ranges) return;
    const int row0 = rg * kRows;
    const int Ng = min(kRows, a.N - row0);                      // rows of `out` this group owns

    // ---- Q and (rotary embedding) the positions of its rows: neither needs the scalars below.  Fragment
    // (row tile, k-step) of the staged Q is one lane-ordered 1 KB; a wave brings in every NW-th.  With the
    // rotation a wave takes k-steps t and t + KS/2 together: they hold a lane's pairs.
    constexpr int kQFrags = ROPE ? NQ * KS / 2 : NQ * KS;
    constexpr int kQPer = (kQFrags + NW - 1) / NW;
    const unsigned char *Qb = static_cast<const unsigned char *>(a.q) + ((size_t)bh * a.N + row0) * G::kRowBytes;
    uint4 qreg[kQPer], qreg2[ROPE ? kQPer : 1];
    int qpos[ROPE ? kQPer : 1];
#pragma unroll
    for (int i = 0; i < kQPer; ++i) {
        const int f = min(wave + NW * i, kQFrags - 1);
        const int qt = ROPE ? f / (KS / 2) : f / KS, t = ROPE ? f % (KS / 2) : f % KS;
        const int row = min(qt * 16 + r16, Ng - 1);
        if constexpr (ROPE) qpos[i] = a.position_ids[(size_t)b * a.N + row0 + row];
        qreg[i] = ldg16(Qb + row * G::kRowBytes + (4 * t + g) * 16);
        if constexpr (ROPE) qreg2[i] = ldg16(Qb + row * G::kRowBytes + (4 * (t + KS / 2) + g) * 16);
    }

    const int P = clampi(P_all - row0, 0, kRows);
    // a packed row sees no packed key beyond itself (the mask is lower triangular)
    const int tree_end = min(P_all, row0 + kRows);

    // ---- this workgroup's tiles.  The tiles of a head are dealt in whole blocks of NW to as few of its
    // `ranges` workgroups as cover them; the others have nothing to do and nobody waits for them.
    const int nA = (C + 31) >> 5;
    const int nT = P > 0 ? nA + ((tree_end + 31) >> 5) : 0;
    const int nblk = (nT + NW - 1) / NW;
    const int per = ranges == 1 ? max(nblk, 1) : max((nblk + ranges - 1) / ranges, 1);
    const int n_part = ranges == 1 ? 1 : max((nblk + per - 1) / per, 1);
    if (split >= n_part) return;
    const int tile_begin = split * per * NW;
    const int tile_end = min(nT, tile_begin + per * NW);
    const int nb = (tile_end - tile_begin + NW - 1) / NW;       // blocks
    const int head = bh - b * a.H;
    // context rows (paged: the pool), and how far from them the packed rows lie: addresses as numbers, because
    // a choice between two captured pointers makes the compiler keep everything that is captured in memory
    const uintptr_t Kc = reinterpret_cast<uintptr_t>(a.k_cache) + (PAGED ? 0 : (size_t)bh * a.Cmax * G::kRowBytes);
    const uintptr_t Vc = reinterpret_cast<uintptr_t>(a.v_cache) + (PAGED ? 0 : (size_t)bh * a.Cmax * G::kRowBytes);
    const uintptr_t Kn = reinterpret_cast<uintptr_t>(a.k_new) + (size_t)bh * a.N * G::kRowBytes - Kc;
    const uintptr_t Vn = reinterpret_cast<uintptr_t>(a.v_new) + (size_t)bh * a.N * G::kRowBytes - Vc;

    const int t_first = tile_begin + wave;
    // this wave's first packed-key tile (it may lie past the end)
    const int tree_first = t_first >= nA ? t_first : t_first + (nA - t_first + NW - 1) / NW * NW;

    // Rows past the end of a tile's keys are redirected to its last key (their probabilities are zero).
    // Page of a tile: through the scalar cache (constant address space; nothing in the kernel writes the table).  As a
    // plain load the compiler makes it a vector load, because of the stores before it, and the wait on that is a wait
    // for every K and V load in flight, once a block (B=8, H=32, C=1024-2048, pages of 64: 56.5 us against 46.8; dense 46.1).
    typedef const __attribute__((address_space(4))) int32_t cint32;
    auto page_of = [&](int tile) __attribute__((always_inline)) {
        const int pg = min(tile * 32 / a.page_size, a.max_pages - 1);
        return clampi(((cint32 *)(uintptr_t)a.block_table)[(size_t)b * a.max_pages + pg], 0, a.n_pages - 1);
    };
    int pid = 0;              // page of the tile that is fetched next (paged context tiles only)
    auto tile_off = [&](int tile, bool tree) __attribute__((always_inline)) -> size_t {   // of the tile's first key
        const uint32_t dense = (uint32_t)(tile - (tree ? nA : 0)) * 32;
        if (!PAGED) return (size_t)dense * G::kRowBytes;
        const size_t paged = ((size_t)pid * a.H + head) * a.page_size + (uint32_t)(tile * 32) % (uint32_t)a.page_size;
        return (tree ? dense : paged) * G::kRowBytes;
    };
    auto tile_keys = [&](int tile, bool tree) __attribute__((always_inline)) {
        return min(32, tree ? tree_end - (tile - nA) * 32 : C - tile * 32);
    };
    vec8 kreg[2][KS], vreg[G::kLoads];                          // (native vectors stay in registers)
    typedef const __attribute__((address_space(1))) vec8 gvec8;   // an address made from a number is a global one
    auto load_k = [&](uintptr_t p, int keys, int ln) __attribute__((always_inline)) {
        if constexpr (kStageK) {          // whole rows
            const uint32_t off0 = (uint32_t)ln * 16, last = (uint32_t)(keys - 1) * G::kRowBytes + (ln % G::kChunks) * 16;
#pragma unroll
            for (int s = 0; s < 2 * KS; ++s) kreg[s / KS][s % KS] = *(gvec8 *)(p + min(off0 + s * 1024u, last));
        } else {                          // operand order
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const uint32_t off = (uint32_t)min(mt * 16 + (ln & 15), keys - 1) * G::kRowBytes + (ln >> 4) * 16;
#pragma unroll
                for (int t = 0; t < KS; ++t) kreg[mt][t] = *(gvec8 *)(p + off + t * 64);
            }
        }
    };
    auto load_v = [&](uintptr_t p, int keys, int ln) __attribute__((always_inline)) {
        const uint32_t off0 = (uint32_t)ln * 16, last = (uint32_t)(keys - 1) * G::kRowBytes + (ln % G::kChunks) * 16;
#pragma unroll
        for (int s = 0; s < G::kLoads; ++s) vreg[s] = *(gvec8 *)(p + min(off0 + s * 1024u, last));
    };

    // ---- rotary embedding of Q: cosines and sines are fetched ahead of K and V, as the wait on them is
    // a wait on everything fetched before
    float qcs[ROPE ? kQPer : 1][8], qsn[ROPE ? kQPer : 1][8];
    if constexpr (ROPE) {
#pragma unroll
        for (int i = 0; i < kQPer; ++i) {
            const int f = min(wave + NW * i, kQFrags - 1), t = f % (KS / 2);
            const size_t o = (size_t)clampi(qpos[i], 0, a.max_pos - 1) * (D / 2) + (4 * t + g) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) { qcs[i][e] = a.cos_tab[o + e]; qsn[i][e] = a.sin_tab[o + e]; }
        }
    }
    // visibility words of the wave's packed-key tiles, and (rotation) the positions of the first one's keys
    uint64_t mword[TB][NQ];
    int kpos[2] = {0, 0};
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const int word = min((tree_first - nA + t * NW) >> 1, a.words - 1);
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt)
            mword[t][qt] = a.mask_bits[((size_t)b * a.N + min(row0 + qt * 16 + r16, a.N - 1)) * a.words + word];
    }
    if constexpr (ROPE) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
            kpos[mt] = a.position_ids[(size_t)b * a.N + clampi((tree_first - nA) * 32 + mt * 16 + r16, 0, max(tree_end - 1, 0))];
    }
    // K and V of this wave's tile of a block.  A wave whose turn falls past the end takes the last tile again
    // (masked: no branch around the loads, which would turn every wait into a wait for all of them); a
    // workgroup without tiles reads the first tile there is and ignores it.
    auto fetch = [&](int tile, int ln, auto which_k, auto which_v) __attribute__((always_inline)) {
        const int tl = max(min(tile, tile_end - 1), 0);
        const bool tree = tl >= nA;
        const size_t off = tile_off(tl, tree);
        const int keys = max(tile_keys(tl, tree), 1);
        if (decltype(which_k)::value) load_k(Kc + off + (tree ? Kn : 0), keys, ln);
        if (decltype(which_v)::value) load_v(Vc + off + (tree ? Vn : 0), keys, ln);
    };
    auto next_page = [&](int tile) __attribute__((always_inline)) {             // looked up one block ahead
        const int tl = max(min(tile, tile_end - 1), 0);
        return PAGED && tl < nA ? page_of(tl) : pid;
    };
    pid = next_page(t_first);
    fetch(t_first, lane, std::true_type{}, std::true_type{});
    pid = next_page(t_first + NW);

    // ---- Q -> LDS
#pragma unroll
    for (int i = 0; i < kQPer; ++i) {
        const int f = wave + NW * i;
        if (f < kQFrags) {
            const int qt = ROPE ? f / (KS / 2) : f / KS, t = ROPE ? f % (KS / 2) : f % KS;
            const bool real = qt * 16 + r16 < P;
            uint4 lo = qreg[i];
            if constexpr (ROPE) {
                lo = rope8<T>(qreg[i], qreg2[i], qcs[i], qsn[i], true);
                uint4 hi = rope8<T>(qreg2[i], qreg[i], qcs[i], qsn[i], false);
                *reinterpret_cast<uint4 *>(sQ + ((qt * KS + t + KS / 2) * 64 + lane) * 16) = real ? hi : make_uint4(0, 0, 0, 0);
            }
            *reinterpret_cast<uint4 *>(sQ + ((qt * KS + t) * 64 + lane) * 16) = real ? lo : make_uint4(0, 0, 0, 0);
        }
    }
    // element (mt, i) of a lane's scores of the t-th packed-key tile = key 16*mt+4g+i: bit 4*mt+i of byte t
    uint32_t vis[NQ];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
        uint32_t packed = 0;
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const uint32_t v32 = (uint32_t)(mword[t][qt] >> (((tree_first - nA + t * NW) & 1) * 32));
            packed |= (((v32 >> (4 * g)) & 0xfu) | (((v32 >> (16 + 4 * g)) & 0xfu) << 4)) << (8 * t);
        }
        vis[qt] = qt * 16 + r16 < P ? packed : 0u;
        if (kVisInLds) {                               // (a lane reads back what it wrote)
#pragma unroll
            for (int t = 0; t < TB; ++t) sVis[((t * NW + wave) * NQ + qt) * 64 + lane] = (unsigned char)(vis[qt] >> (8 * t));
        } else asm volatile("" : "+v"(vis[qt]));         // computed here, not sunk into the loop's masked path
    }

    // this wave's part of the output: row tiles RW*i + q_first, d-tiles j_first ..
    const int j_first = RW > 1 ? wave % DT : wave * JW, q_first = RW > 1 ? wave / DT : 0;
    unsigned char *my_tile = sV + wave * G::kTileBytes;
    auto v_wr = [&](int s, int ln) __attribute__((always_inline)) {
        const int row = ln / G::kChunks, base = row * G::kRowBytes + vswz<D>(row, ln % G::kChunks) * 16;
        return s * 1024 + (base ^ (((s * G::kRowsPerLoad) & (G::kChunks / 2 - 1)) * 32));
    };
    auto vt_rd = [&](int dt, int ln) __attribute__((always_inline)) {
        const int r = ln & 15, row = 4 * (ln >> 4) + (r >> 2);
        const int base = row * G::kRowBytes + vswz<D>(row, (r & 3) >> 1) * 16 + (r & 1) * 8;
        return base ^ ((dt & (G::kChunks / 2 - 1)) * 32);
    };

    lds_barrier();            // Q visible to all waves
    RD_TR(1);

    // rows -> operand order, 16 keys at a time through the wave's own piece of LDS
    auto turn_k = [&](int ln) __attribute__((always_inline)) {
        if constexpr (kStageK) {
            unsigned char *st = sK + wave * (16 * G::kRowBytes);
            const int row = ln / G::kChunks, wr = row * G::kRowBytes + kswz<D>(row, ln % G::kChunks) * 16;
            const int rd = (ln & 15) * G::kRowBytes + kswz<D>(ln & 15, ln >> 4) * 16;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    *reinterpret_cast<vec8 *>(st + s * 1024 + (wr ^ (((s * G::kRowsPerLoad) & (G::kChunks - 1)) * 16))) = kreg[mt][s];
                wave_lds_sync();
#pragma unroll
                for (int t = 0; t < KS; ++t) kreg[mt][t] = *reinterpret_cast<const vec8 *>(st + (rd ^ ((4 * t & (G::kChunks - 1)) * 16)));
                wave_lds_sync();
            }
        }
    };

    const int nqt = (P + 15) >> 4;
    const float c_abs = fabsf(a.scale_log2e);
    const bool c_neg = a.scale_log2e < 0.f;

    // One block; `more`: there is another one, whose K and V are fetched here.
    auto block_step = [&](auto nqa_tag, auto more_tag, int ib, const vec8 (&qf)[kQReg ? NQ : 1][KS], auto &m_ref, auto &l_own, auto &oacc, auto &m_out, auto &l_out) __attribute__((always_inline)) {
        constexpr int NQA = decltype(nqa_tag)::value;
        constexpr bool more = decltype(more_tag)::value;
        // lane numbers through an opaque copy: addresses derived from them are made anew in each block (one or two
        // operations) and not kept in registers across the loop, where the larger instances would park them in
        // scratch memory and wait for ALL loads in flight on every reload
        int lane = tid & 63;
        if (NQA * JW >= 3) asm volatile("" : "+v"(lane));
        const int r16 = lane & 15, g = lane >> 4;
        const int tile = t_first + ib * NW;
        const bool tree = tile >= nA;
        turn_k(lane);
        if constexpr (ROPE) {
            if (tree && tile < tile_end) {       // packed keys: rotated here; the rotated rows also go to a.k_rot (what a cache stores)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const int key = (tile - nA) * 32 + mt * 16 + r16;
                    int pos = kpos[mt];
                    if (tile != tree_first) pos = a.position_ids[(size_t)b * a.N + min(key, tree_end - 1)];
                    const size_t o = (size_t)clampi(pos, 0, a.max_pos - 1) * (D / 2) + g * 8;
#pragma unroll
                    for (int t = 0; t < KS / 2; ++t) {
                        float cs[8], sn[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) { cs[e] = a.cos_tab[o + t * 32 + e]; sn[e] = a.sin_tab[o + t * 32 + e]; }
                        const uint4 lo = __builtin_bit_cast(uint4, kreg[mt][t]), hi = __builtin_bit_cast(uint4, kreg[mt][t + KS / 2]);
                        kreg[mt][t] = __builtin_bit_cast(vec8, rope8<T>(lo, hi, cs, sn, true));
                        kreg[mt][t + KS / 2] = __builtin_bit_cast(vec8, rope8<T>(hi, lo, cs, sn, false));
                        if (a.k_rot != nullptr && key < tree_end) {
                            unsigned char *kr = static_cast<unsigned char *>(a.k_rot) + ((size_t)bh * a.N + key) * G::kRowBytes + (4 * t + g) * 16;
                            *reinterpret_cast<vec8 *>(kr) = kreg[mt][t];
                            *reinterpret_cast<vec8 *>(kr + D) = kreg[mt][t + KS / 2];
                        }
                    }
                }
            }
        }
        f32x4 sacc[2][NQA];
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) sacc[0][qt] = sacc[1][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            const vec8 a0 = kreg[0][t], a1 = kreg[1][t];
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                const vec8 bq = kQReg ? qf[kQReg ? qt : 0][t] : *reinterpret_cast<const vec8 *>(sQ + ((qt * KS + t) * 64 + lane) * 16);
                sacc[0][qt] = Elem<T>::mfma(a0, bq, sacc[0][qt]);
                sacc[1][qt] = Elem<T>::mfma(a1, bq, sacc[1][qt]);
            }
        }
        if (NQA * JW > 3) __builtin_amdgcn_sched_barrier(0);      // K's registers are read before they are fetched again
        int pid_next = pid;
        if (more) {
            fetch(tile + NW, lane, std::true_type{}, std::false_type{});
            pid_next = next_page(tile + 2 * NW);                // (behind the softmax by the time it is waited for)
        }

        // softmax in log2 units.  An interior context tile keeps the raw scores (the scale is folded into
        // the exponent); a tile with masked or missing keys is scaled here and its dead entries set to -inf.
        const int rem = tile < tile_end ? tile_keys(tile, tree) : 0;
        const bool plain = !tree && rem >= 32 && !c_neg;
        float mx[NQA];
        if (plain) {
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt)
                mx[qt] = quad_max(fmaxf(fmaxf(fmaxf(sacc[0][qt][0], sacc[0][qt][1]), fmaxf(sacc[0][qt][2], sacc[0][qt][3])),
                                        fmaxf(fmaxf(sacc[1][qt][0], sacc[1][qt][1]), fmaxf(sacc[1][qt][2], sacc[1][qt][3])))) * c_abs;
        } else {
            const uint32_t tail = rem >= 32 ? 0xffffffffu : (rem <= 0 ? 0u : ((1u << rem) - 1u));
            const uint32_t tail8 = ((tail >> (4 * g)) & 0xfu) | (((tail >> (16 + 4 * g)) & 0xfu) << 4);
            const int tb = tree ? (tile - tree_first) / NW : 0;
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                const uint32_t vq = kVisInLds ? sVis[((tb * NW + wave) * NQ + qt) * 64 + lane] : vis[qt] >> (8 * tb);
                const uint32_t bits = (tree ? vq : 0xffu) & tail8;
                float tmax = -INFINITY;
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float sv = ((bits >> (4 * mt + i)) & 1u) ? sacc[mt][qt][i] * a.scale_log2e : -INFINITY;
                        sacc[mt][qt][i] = sv;
                        tmax = fmaxf(tmax, sv);
                    }
                mx[qt] = quad_max(tmax);
            }
        }
        const float c_fold = plain ? c_abs : 1.0f;
        // Reference of the exponents: the workgroup's running one, or this tile's maximum in rows where it lies
        // more than 2^kSlack above that.  Rows seldom move once the first block is in, and while none does
        // (`moved`, agreed through LDS) the products add up without a factor.
        float ref[NQA], psum[NQA];
        vec8 pb[NQA];
        bool moved = false;
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) {
            const bool up = mx[qt] > m_ref[qt] + kSlack;
            moved |= __builtin_amdgcn_ballot_w64(up) != 0;
            ref[qt] = up ? mx[qt] : m_ref[qt];
            const float m_safe = (ref[qt] == -INFINITY) ? 0.f : ref[qt];
            float sum = 0.f;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[mt][qt][i], c_fold, -m_safe));
                    sum += pv;
                    pb[qt][4 * mt + i] = (T)pv;
                }
            psum[qt] = sum;
            // the last block's table also carries the waves' sums
            if (!more) psum[qt] = quad_sum(l_own[qt] * __builtin_amdgcn_exp2f(m_ref[qt] - m_safe) + sum);
        }
        if (ib > 0) lds_barrier();        // the block before is read
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt)
            *reinterpret_cast<vec8 *>(sP + ((wave * NQ + qt) * 64 + lane) * 16) = pb[qt];
        if (!more || moved) {
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt)
                if (g == 0) *reinterpret_cast<float2 *>(sML + (qt * 16 + r16) * kMLStride + wave * 8) = make_float2(ref[qt], psum[qt]);
        }
        if (more && lane == 0) sMoved[wave] = moved ? 1 : 0;
#pragma unroll
        for (int s = 0; s < G::kLoads; ++s) *reinterpret_cast<vec8 *>(my_tile + v_wr(s, lane)) = vreg[s];
        if (NQA * JW > 3) __builtin_amdgcn_sched_barrier(0);
        if (more) {
            fetch(tile + NW, lane, std::false_type{}, std::true_type{});
            pid = pid_next;
        }
        lds_barrier();                    // tiles, probabilities and references of all waves visible

        constexpr int QWA = (NQA + RW - 1) / RW;
        auto row_tile = [&](int i) __attribute__((always_inline)) { return RW == 1 ? i : min(RW * i + q_first, NQA - 1); };
        auto v_frag = [&](int kt, int j) __attribute__((always_inline)) {
            const unsigned char *vt = sV + kt * G::kTileBytes + vt_rd(j_first + j, lane);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)vt);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(vt + 16 * G::kRowBytes));
            return __builtin_bit_cast(vec8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto p_frag = [&](int kt, int qt) __attribute__((always_inline)) { return *reinterpret_cast<const vec8 *>(sP + ((kt * NQ + qt) * 64 + lane) * 16); };
        uint32_t any = 1;
        int4 mv[NW / 4];
        if (more) {
            any = 0;
#pragma unroll
            for (int w = 0; w < NW / 4; ++w) {
                mv[w] = *reinterpret_cast<const int4 *>(sMoved + 4 * w);
                any |= mv[w].x | mv[w].y | mv[w].z | mv[w].w;
            }
            any = __builtin_amdgcn_readfirstlane(any);
        }
        if (any == 0) {
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) l_own[qt] += psum[qt];
#pragma unroll
            for (int kt = 0; kt < NW; ++kt) {
                vec8 aV[JW];
#pragma unroll
                for (int j = 0; j < JW; ++j) aV[j] = v_frag(kt, j);
#pragma unroll
                for (int i = 0; i < QWA; ++i) {
                    const vec8 pB = p_frag(kt, row_tile(i));
#pragma unroll
                    for (int j = 0; j < JW; ++j) oacc[i][j] = Elem<T>::mfma(aV[j], pB, oacc[i][j]);
                }
                if (NQA * JW > 2) __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        // some row's reference moves (or the sums are due): products scaled by 2^(tile reference - new reference)
        constexpr int QP = QWA * JW > 3 ? (QWA + 1) / 2 : QWA;       // row tiles per pass over V: the factors of more of them do not fit
        const int n_here = tile_end - (tile - wave);            // tiles of this block (those past the end hold zeros)
        float m_new[NQA];
#pragma unroll
        for (int i0 = 0; i0 < QWA; i0 += QP) {
            float fac[QP][NW];
#pragma unroll
            for (int i = 0; i < QP; ++i) {
                if (i0 + i >= QWA) continue;
                const int qt = row_tile(i0 + i);
                float m_old = m_ref[RW == 1 ? i0 + i : 0];
                if (RW > 1) {
#pragma unroll
                    for (int q = 1; q < NQA; ++q) m_old = q == qt ? m_ref[q] : m_old;
                }
                f32x4 ml[NW / 2];
#pragma unroll
                for (int w = 0; w < NW / 2; ++w) ml[w] = *reinterpret_cast<const f32x4 *>(sML + (qt * 16 + r16) * kMLStride + w * 16);
                float m = m_old;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    if (more) {
                        const int f = w % 4 == 0 ? mv[w / 4].x : w % 4 == 1 ? mv[w / 4].y : w % 4 == 2 ? mv[w / 4].z : mv[w / 4].w;
                        ml[w / 2][2 * (w & 1)] = f ? ml[w / 2][2 * (w & 1)] : m_old;
                    }
                    m = fmaxf(m, ml[w / 2][2 * (w & 1)]);
                }
                const float m_safe = (m == -INFINITY) ? 0.f : m;
                float l = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    fac[i][w] = __builtin_amdgcn_exp2f(ml[w / 2][2 * (w & 1)] - m_safe);
                    if (!more) l += fac[i][w] * ml[w / 2][2 * (w & 1) + 1];
                }
                const float alpha = __builtin_amdgcn_exp2f(m_old - m_safe);
#pragma unroll
                for (int j = 0; j < JW; ++j) oacc[i0 + i][j] *= alpha;
                if (!more) { m_out[i0 + i] = m; l_out[i0 + i] = l; }
                if (RW == 1) m_new[i0 + i] = m;
            }
            auto pv_tile = [&](int kt) __attribute__((always_inline)) {
                vec8 aV[JW];
#pragma unroll
                for (int j = 0; j < JW; ++j) aV[j] = v_frag(kt, j);
#pragma unroll
                for (int i = 0; i < QP; ++i) {
                    if (i0 + i >= QWA) continue;
                    const vec8 pB = p_frag(kt, row_tile(i0 + i));
#pragma unroll
                    for (int j = 0; j < JW; ++j)
                        oacc[i0 + i][j] += fac[i][kt] * Elem<T>::mfma(aV[j], pB, f32x4{0.f, 0.f, 0.f, 0.f});
                }
            };
#pragma unroll
            for (int kt = 0; kt < NW / 2; ++kt) { pv_tile(kt); __builtin_amdgcn_sched_barrier(0); }
            if (n_here > NW / 2) {
#pragma unroll
                for (int kt = NW / 2; kt < NW; ++kt) { pv_tile(kt); __builtin_amdgcn_sched_barrier(0); }
            }
        }
        if (more) {
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                float m = m_ref[qt];
                if (RW == 1) {
                    m = m_new[qt];
                } else {
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const int f = w % 4 == 0 ? mv[w / 4].x : w % 4 == 1 ? mv[w / 4].y : w % 4 == 2 ? mv[w / 4].z : mv[w / 4].w;
                        const float r = *reinterpret_cast<const float *>(sML + (qt * 16 + r16) * kMLStride + w * 8);
                        m = fmaxf(m, f ? r : -INFINITY);
                    }
                }
                const float m_safe = (m == -INFINITY) ? 0.f : m;
                l_own[qt] = l_own[qt] * __builtin_amdgcn_exp2f(m_ref[qt] - m_safe) + psum[qt] * __builtin_amdgcn_exp2f(ref[qt] - m_safe);
                m_ref[qt] = m;
            }
        }
    };
    T *outp = static_cast<T *>(a.out) + ((size_t)bh * a.N + row0) * D;
    auto put = [&](int i, f32x4 (&o)[JW], float l) __attribute__((always_inline)) {
        const int qt = RW * i + q_first, row = qt * 16 + r16;
        if (qt < NQ && row < Ng) {
            const bool keep = row < P;                          // rows beyond the packed count are zero
            const float inv = keep ? 1.0f / l : 0.f;
#pragma unroll
            for (int j = 0; j < JW; ++j) {
                f32x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = keep ? o[j][e] * inv : 0.f;
                    asm volatile("" : "+v"(v));                 // an fp32 product, then one rounding, in every instance
                    y[e] = v;
                }
                store_out4(outp + (size_t)row * D + (j_first + j) * 16 + 4 * g, y[0], y[1], y[2], y[3]);
            }
        }
    };
    auto finish = [&](auto nqa_tag, auto &m_run, auto &l_run, auto &oacc) __attribute__((always_inline)) {
    constexpr int QWA = (decltype(nqa_tag)::value + RW - 1) / RW;      // row tiles that can hold packed rows; the rest of the output is zero
    if (n_part == 1) {        // the head's only workgroup
#pragma unroll
        for (int i = 0; i < QW; ++i) put(i, oacc[i < QWA ? i : 0], l_run[i < QWA ? i : 0]);
        RD_TR(6);
        return;
    }

    // ---- partial state -> workspace; the last workgroup of this head (and row group) merges -----------
    // Layout of one partial: (m, l) per row, then the fragments [row tile][d-tile][64 lanes][4], so that
    // every wave store and load covers 1 KB.
    const size_t unit = (size_t)bh * n_rg + rg;
    float *part = a.partials + ((size_t)bh * a.S + split * n_act + rg) * kPF;
    auto frag = [&](int i, int j) __attribute__((always_inline)) { return 2 * kRows + (((RW * i + q_first) * DT + j_first + j) * 64 + lane) * 4; };
    auto real = [&](int i) __attribute__((always_inline)) { return RW * i + q_first < NQ && (RW * i + q_first) * 16 + r16 < P; };
#pragma unroll
    for (int i = 0; i < QWA; ++i) {
        if (real(i)) {
            if (j_first == 0 && g == 0) st_dev2(part + 2 * ((RW * i + q_first) * 16 + r16), m_run[i], l_run[i]);
#pragma unroll
            for (int j = 0; j < JW; ++j) st_dev4(part + frag(i, j), oacc[i][j][0], oacc[i][j][1], oacc[i][j][2], oacc[i][j][3]);
        }
    }
    RD_TR(4);
    const int last = arrive_is_last(a.counters + unit, (uint32_t)n_part);
    RD_TR(5);
    if (last == kNotLast) return;
    const bool cached = (last == kLastClean);
    // (the fp32 kernel merges alike, but as a function of both this moves registers about and costs 1 % at five row tiles)
    constexpr int kChunk = 6;                                   // partials whose loads are in flight together
    constexpr int kPair = QWA < 2 || JW > 1 ? 1 : 2;                       // row tiles merged together
    const float *hp = a.partials + ((size_t)bh * a.S + rg) * kPF;
#pragma unroll
    for (int i0 = 0; i0 < QW; i0 += kPair) {
        float M[kPair], den[kPair];
        f32x4 acc[kPair][JW];
#pragma unroll
        for (int u = 0; u < kPair; ++u) {
            M[u] = -INFINITY;
            den[u] = 0.f;
#pragma unroll
            for (int j = 0; j < JW; ++j) acc[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (i0 < QWA && (RW * i0 + q_first) * 16 < P) {
#pragma unroll 1
            for (int s0 = 0; s0 < n_part; s0 += kChunk) {
                float2 ml[kPair][kChunk];
                f32x4 fr[kPair][kChunk][JW];
#pragma unroll
                for (int c = 0; c < kChunk; ++c) {
                    const bool have = s0 + c < n_part;          // uniform
                    const float *ps = hp + (size_t)(s0 + c) * n_act * kPF;
#pragma unroll
                    for (int u = 0; u < kPair; ++u) {
                        ml[u][c] = make_float2(-INFINITY, 0.f); // absent: weight 2^-inf = 0
#pragma unroll
                        for (int j = 0; j < JW; ++j) fr[u][c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (have && i0 + u < QWA && real(i0 + u)) {
                            const float *pm = ps + 2 * ((RW * (i0 + u) + q_first) * 16 + r16);
                            if (cached) {
                                ml[u][c] = *reinterpret_cast<const float2 *>(pm);
#pragma unroll
                                for (int j = 0; j < JW; ++j) fr[u][c][j] = *reinterpret_cast<const f32x4 *>(ps + frag(i0 + u, j));
                            } else {
                                ml[u][c] = ld_dev2(pm);
#pragma unroll
                                for (int j = 0; j < JW; ++j) {
                                    const float2 lo = ld_dev2(ps + frag(i0 + u, j)), hi = ld_dev2(ps + frag(i0 + u, j) + 2);
                                    fr[u][c][j] = f32x4{lo.x, lo.y, hi.x, hi.y};
                                }
                            }
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < kPair; ++u) {
                    float Mn = M[u];
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) Mn = fmaxf(Mn, ml[u][c].x);
                    const float Ms = (Mn == -INFINITY) ? 0.f : Mn;
                    const float resc = __builtin_amdgcn_exp2f(M[u] - Ms);
                    den[u] *= resc;
#pragma unroll
                    for (int j = 0; j < JW; ++j) acc[u][j] *= resc;
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) {
                        const float w = __builtin_amdgcn_exp2f(ml[u][c].x - Ms);
                        den[u] += w * ml[u][c].y;
#pragma unroll
                        for (int j = 0; j < JW; ++j) acc[u][j] += w * fr[u][c][j];
                    }
                    M[u] = Mn;
                }
            }
        }
        RD_TR(7);
#pragma unroll
        for (int u = 0; u < kPair; ++u)
            if (i0 + u < QW) put(i0 + u, acc[u], den[u]);
    }
    if (tid == 0) a.counters[unit] = 0;   // leave the workspace ready for the next call
    RD_TR(6);
    };

    // Loop and epilogue are instantiated for all row tiles and for the lower half (a padded row tile costs as
    // much as a real one); the last block, which fetches nothing, is a step of its own.
    auto walk = [&](auto nqa_tag) __attribute__((always_inline)) {
        constexpr int NQA = decltype(nqa_tag)::value;
        constexpr int QWA = (NQA + RW - 1) / RW;
        float m_ref[NQA], l_own[NQA];     // exponents' reference of every row; this wave's share of the sums (lane partials)
        float m_run[QWA], l_run[QWA];     // in the end: reference and sum of the rows this wave writes
        f32x4 oacc[QWA][JW];
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) { m_ref[qt] = -INFINITY; l_own[qt] = 0.f; }
#pragma unroll
        for (int i = 0; i < QWA; ++i) {
            m_run[i] = -INFINITY;
            l_run[i] = 0.f;
#pragma unroll
            for (int j = 0; j < JW; ++j) oacc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        vec8 qf[kQReg ? NQ : 1][KS];
        if constexpr (kQReg) {
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt)
#pragma unroll
                for (int t = 0; t < KS; ++t) qf[qt][t] = *reinterpret_cast<const vec8 *>(sQ + ((qt * KS + t) * 64 + lane) * 16);
        }
        for (int ib = 0; ib + 1 < nb; ++ib) block_step(nqa_tag, std::true_type{}, ib, qf, m_ref, l_own, oacc, m_run, l_run);
        if (nb > 0) block_step(nqa_tag, std::false_type{}, nb - 1, qf, m_ref, l_own, oacc, m_run, l_run);
        RD_TR(3);
        finish(nqa_tag, m_run, l_run, oacc);
    };
    constexpr int kHalf = (NQ + 1) / 2;
    if (NQ > 1 && nqt <= kHalf) walk(std::integral_constant<int, kHalf>{});
    else walk(std::integral_constant<int, NQ>{});

}

template <int D, int NQ, int NW, int TB>
static constexpr size_t mfma_smem_bytes()
{
    return (size_t)NQ * Geo<D>::kKSteps * 1024 + (size_t)NW * Geo<D>::kTileBytes + (size_t)NW * NQ * 1024 + (size_t)NQ * 16 * (NW * 8 + 16) + NW * sizeof(int) +
           (NQ > 4 ? (size_t)TB * NW * NQ * 64 : 0) + (stage_k<D, NQ, NW>() ? (size_t)NW * 16 * Geo<D>::kRowBytes : 0);
}

template <typename T, int D, int NQ, int NW, int TB, bool PAGED, bool ROPE>
static int launch_mfma(const AttnArgs &a, hipStream_t stream)
{
    constexpr size_t smem = mfma_smem_bytes<D, NQ, NW, TB>();
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    static std::atomic<unsigned long long> configured{0};
    const int st = ensure_dynamic_lds(reinterpret_cast<const void *>(&rd_tree_attn_mfma_kernel<T, D, NQ, NW, TB, PAGED, ROPE>), smem, configured);
    if (st != RD_OK) return st;
    const size_t wgs = ((size_t)a.B * a.H + 7) / 8 * 8 * a.S;
    if (wgs > 0x7fffffffull) return RD_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((rd_tree_attn_mfma_kernel<T, D, NQ, NW, TB, PAGED, ROPE>), dim3((unsigned)wgs), dim3(NW * 64), smem, stream, a);
    return rd_check_launch();
}

template <typename T, int D, int NW, bool PAGED, bool ROPE>
static int dispatch_nq(const AttnArgs &a, int rg_tiles, hipStream_t stream)
{
    const int tb = ((a.N + 31) / 32 + NW - 1) / NW;             // packed-key tiles a wave can meet
    if (tb > 1) {                                               // (N > 32 NW: the largest row groups)
        if (rg_tiles != kGroupTiles) return RD_ERR_UNSUPPORTED;
        if (tb == 2) return launch_mfma<T, D, kGroupTiles, NW, 2, PAGED, ROPE>(a, stream);
        if constexpr (NW == 4) {
            if (tb == 3) return launch_mfma<T, D, kGroupTiles, 4, 3, PAGED, ROPE>(a, stream);
        }
        return RD_ERR_UNSUPPORTED;
    }
    switch (rg_tiles) {
    case 1: return launch_mfma<T, D, 1, NW, 1, PAGED, ROPE>(a, stream);
    case 2: return launch_mfma<T, D, 2, NW, 1, PAGED, ROPE>(a, stream);
    case 3: return launch_mfma<T, D, 3, NW, 1, PAGED, ROPE>(a, stream);
    case 4: return launch_mfma<T, D, 4, NW, 1, PAGED, ROPE>(a, stream);
    case 5: return launch_mfma<T, D, 5, NW, 1, PAGED, ROPE>(a, stream);
    default: return RD_ERR_UNSUPPORTED;
    }
}

template <typename T, bool PAGED, bool ROPE = false>
static int tree_attn_mfma(const AttnArgs &a, int D, int waves, int rg_tiles, hipStream_t stream)
{
    if (D == 128)
        return waves == 8 ? dispatch_nq<T, 128, 8, PAGED, ROPE>(a, rg_tiles, stream) : dispatch_nq<T, 128, 4, PAGED, ROPE>(a, rg_tiles, stream);
    return waves == 8 ? dispatch_nq<T, 64, 8, PAGED, ROPE>(a, rg_tiles, stream) : dispatch_nq<T, 64, 4, PAGED, ROPE>(a, rg_tiles, stream);
}

}  // namespace rd
