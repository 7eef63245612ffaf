// Tree-masked attention of the packed candidates against the KV cache (Sec. 3.3, 3.4) on the gfx950 matrix cores
// for 16-bit K/V (bf16 or fp16): a split-key flash kernel, its template and dispatch, instantiated per element
// type, cache layout and rotation (rd_tree_attn_bf16.hip, _f16, _paged, _rope_bf16, _rope_f16).
//
// A key range is a sequence of 32-key tiles, the context's first, then the packed keys'.  Waves take tiles in turn, and no
// wave waits for another while they last.  Per tile a wave
//   * has K and V copied from memory straight into its own piece of LDS (16 KB at D = 128; the next tile's K is on its
//     way as soon as this one's is in registers, the same for V);
//   * forms S^T = K Q^T with K as the A operand and Q, shared by the workgroup in LDS, as the B operand;
//   * takes the softmax of its 32 keys (keys taken as 4g+i, 16+4g+i: the probabilities its lanes hold are then the B
//     operand of the next product) and adds to its own O^T = V^T P^T, V^T read by transpose reads.
// In the end the waves' states meet in LDS.  A range of at most one tile per wave takes a shorter way: every wave adds up a
// share of the output over all the tiles.
//
// What bounds it.  Long contexts in large batches: HBM; the same copies without any arithmetic take as long (B=16, H=64,
// C=2048 192 us, 5.6 TB/s; 191 without arithmetic).  Few heads: a chain of latencies (counts, Q, K and V in 4.4 us at H=32,
// C=1024, 2.3 of arithmetic, the store of a partial result and its arrival 1.4, the merge 2.3), in which a branch per tile, a
// half-written line and a load that only fills a chunk all count: the sum over the tiles without branches, partial results
// stored 16 bytes at a time and merged by chunks of 4, 6 or 8 take H=32, C=1024 from 11.6 to 11.0 us, with rotation from 12.5 to
// 12.0, H=32, C=1777, 209 rows of 350 from 26.2 to 24.8.  Several row groups: the copies, of which a compute unit has some 48 KB
// under way at most, 21 bytes a clock from beyond L2, and every group of a range waits for the same ones (taking the tiles in
// another order in each group, so that most are in L2, is slower: 23.2 us against 21.4).  A wave's own chain of a tile, beside that:
// Q's operands read ahead and V's before the exponents shorten it (scores 1280 -> 500 clocks of 3380), H=32, C=1024 by 1 %.  Against the kernel it
// replaced, whose waves shared every block of tiles at two barriers and fetched K and V through registers, us per launch, K
// and V from memory: H=32, C=1024 12.1 -> 10.8; B=4, H=32, C=1024 23.9 -> 19.6; H=32, C=1777, 61 rows 22.3 -> 16.7 and 147
// rows 30.0 -> 22.0; B=10, H=52, C=63-92, 207 tokens 49.4 -> 33.2; B=4, H=40, C=4096 74.5 -> 66.5; B=16, H=52, C=2048 183.5 ->
// 178; B=24, H=32, C=101-1500, 25 tokens, bf16 in a dense cache 78.3 -> 69.3; nothing at B=9, H=26, C=5384 (106.7 -> 106.3).
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

// Floats between rows of the waves' statistics: eight waves' 16 rows in distinct banks.  (Four waves and three row tiles: with
// more than four floats a row the second workgroup does not fit the compute unit's LDS.)
constexpr int stat_stride(int waves) { return waves == 8 ? 12 : 4; }

// NW = waves per workgroup (4 or 8); NQ = row tiles (16 packed rows).
// PAGED: the context keys and values live in fixed-size pages found through a block table
// (a.block_table, a.page_size, a.max_pages) instead of one dense [B,H,Cmax,D] tensor.
// ROPE: q and k_new arrive unrotated; the kernel applies the rotary embedding at a.position_ids
// to the query rows as it brings them into LDS and to the packed-key tiles as it walks them.
// ALL: a workgroup takes all row groups of a head, one after the other (one key range each).
template <typename T, int D, int NQ, int NW, bool PAGED, bool ROPE, bool ALL>
__global__ __launch_bounds__(NW * 64, 2) void rd_tree_attn_mfma_kernel(AttnArgs a)
{
    using G = Geo<D>;
    using vec8 = typename Elem<T>::vec8;
    constexpr int KS = G::kKSteps;
    constexpr int DT = G::kDTiles;
    constexpr int RB = G::kRowBytes;
    constexpr int kLoads = G::kLoads;                           // wave loads per tile
    constexpr int kRows = NQ * 16;
    constexpr int kPF = kRows * 2 + DT * NQ * 256;              // floats per partial: (m,l) per row, then fragments
    // Fragments (row tile, d-tile) of the output are shared out to the waves two row tiles at a time, fragment f to wave f % NW.
    constexpr int kRounds = (NQ + 1) / 2, kOwn = 2 * DT / NW;   // a wave's fragments per round
    constexpr int kStat = stat_stride(NW);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *sK = smem;                                   // [NW] K tiles; in the end, with sV, the waves' results
    unsigned char *sV = sK + NW * G::kTileBytes;                // [NW] V tiles
    unsigned char *sQ = sV + NW * G::kTileBytes;                // [kRows] rows
    unsigned char *sMask = sQ + kRows * RB;                     // [NW][64] visibility words of the rows (packed-key tiles)
    float *sM = reinterpret_cast<float *>(sMask + NW * 256);    // [kRows][NW] maxima, rows kStat apart
    float *sL = sM + kRows * kStat;                             // ... and sums
    constexpr float kSlack = 8.f;                               // exponents may exceed their reference by this much

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)smem;
    const uint32_t ldsK = lds0 + wave * G::kTileBytes, ldsV = ldsK + NW * G::kTileBytes;
    const uint32_t ldsQ = lds0 + 2 * NW * G::kTileBytes, ldsMask = ldsQ + kRows * RB + wave * 256;
    RD_TR(0);
    // All arguments are fetched here, together: as the compiler places the loads they are a chain of four, 0.3 us each.
    asm volatile("" : : "s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.k_new), "s"(a.v_new), "s"(a.ctx_len), "s"(a.n_packed), "s"(a.mask_bits),
                 "s"(a.B), "s"(a.H), "s"(a.N), "s"(a.Cmax), "s"(a.S), "s"(a.words), "s"(a.n_rg), "s"(a.ranges), "s"(a.usual), "s"(a.sorted));
    if constexpr (ROPE) asm volatile("" : : "s"(a.position_ids), "s"(a.cos_tab), "s"(a.sin_tab), "s"(a.max_pos));
    if constexpr (PAGED) asm volatile("" : : "s"(a.block_table), "s"(a.page_size), "s"(a.max_pages), "s"(a.n_pages));

    // ---- which (sequence, head), which of its a.S workgroups.  Workgroups are dealt round-robin to the 8 XCDs; all of
    // a head's go to one of them, whose L2 then serves Q, K/V shared by row groups and the partial results (merging
    // partials past the L2 takes about twice as long).  Head numbers past the end fill up the last eight.
    // Lengths come through the scalar cache (constant address space; nothing in the kernel writes them) and are not waited
    // for before the keys are needed.
    typedef const __attribute__((address_space(4))) int32_t cint32;
    cint32 *ctx_len = (cint32 *)(uintptr_t)a.ctx_len, *packed = (cint32 *)(uintptr_t)a.n_packed;
    const int xcd = (int)(blockIdx.x & 7), n_rg = a.n_rg;
    // (ALL has one range, so that its instances hold no merge and its registers: B=1024, H=4, 16 x 5 tokens, C=60 78.5 -> 75.9 us)
    int bh, b, r_wg, n_act = 1, ranges = ALL ? 1 : attn_ranges(a.ranges, 1);      // n_act row groups times ranges: the head's workgroups
    auto groups_of = [&](int rows) __attribute__((always_inline)) { return max((clampi(rows, 0, a.N) + kRows - 1) / kRows, 1); };
    auto heads_before = [&](int s) __attribute__((always_inline)) { return (s * a.H + 7 - xcd) >> 3; };         // this XCD's, of sequences before s
    auto wgs_of = [&](int s, int act) __attribute__((always_inline)) { return (heads_before(s + 1) - heads_before(s)) * act * ranges; };
    auto running = [&](int x) __attribute__((always_inline)) {             // sum over the lanes up to this one
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(x, o, 64);                 // (by all lanes)
            x += lane >= o ? up : 0;
        }
        return x;
    };
    if constexpr (ALL) {                      // one workgroup per head, which takes the row groups one after the other
        bh = (int)(blockIdx.x >> 3) * 8 + xcd;
        if (bh >= a.B * a.H) return;
        b = bh / a.H;
        r_wg = 0;
        n_act = groups_of(packed[b]);
    } else if (n_rg == 1 && !a.sorted) {
        const int k = (int)(blockIdx.x >> 3), hl = ranges == 1 ? k : k / ranges;
        r_wg = k - hl * ranges;
        bh = hl * 8 + xcd;
        if (bh >= a.B * a.H) return;
        b = a.B == 1 ? 0 : bh / a.H;
    } else if (a.B == 1) {                    // only row groups that hold packed rows get workgroups
        n_act = groups_of(packed[0]);
        ranges = attn_ranges(a.ranges, n_act);
        const int k = (int)(blockIdx.x >> 3), n_wg = n_act * ranges, hl = k / n_wg;
        r_wg = k - hl * n_wg;
        bh = hl * 8 + xcd;
        if (bh >= a.H) return;
        b = 0;
    } else {
        // Only row groups that hold packed rows get workgroups, so their number is the sequence's own: a lane counts those of
        // one sequence's heads on this XCD, of four in large batches (a step of 64 costs 0.4 us: 512 sequences, H=32, 20 to 300
        // keys, 80 tokens 680 us by steps of 64, 614 by 256), and a running sum finds the workgroup's place.  (Workgroups without work in between
        // leave compute units idle beside others that have two: 29 us for 22 at H=32, C=1777, 147 of 350 rows.)
        ranges = a.usual;
        int own = (int)(blockIdx.x >> 3);     // in the end: the workgroup's number among its sequence's
        if (a.B <= kOneStep) {                // a sequence to a lane
            int seq = min(lane, a.B - 1), rows = a.n_packed[seq];
            if (a.sorted) {                   // where there are more workgroups than fit the chip at once, those of long sequences first
                const int keys = lane < a.B ? a.ctx_len[seq] : -1;
                int place = 0;
                for (int j = 0; j < a.B; ++j) {
                    const int other = __builtin_amdgcn_readlane(keys, j);
                    place += other > keys || (other == keys && j < lane) ? 1 : 0;
                }
                place = lane < a.B ? place : lane;              // (a permutation of the lanes)
                seq = __builtin_amdgcn_ds_permute(place * 4, seq);
                rows = __builtin_amdgcn_ds_permute(place * 4, rows);
            }
            const int act = groups_of(rows), act0 = __builtin_amdgcn_readlane(act, 0);
            if (__builtin_amdgcn_ballot_w64(act != act0) == 0) ranges = attn_ranges(a.ranges, act0);      // (all sequences alike)
            const int need = lane < a.B ? wgs_of(seq, act) : 0, sum = running(need);
            const uint64_t past = __builtin_amdgcn_ballot_w64(sum > own);
            if (past == 0) return;
            const int at = __builtin_ctzll(past);
            own -= __builtin_amdgcn_readlane(sum, at) - __builtin_amdgcn_readlane(need, at);
            n_act = __builtin_amdgcn_readlane(act, at);
            b = __builtin_amdgcn_readlane(seq, at);
        } else {
            int s0 = 0, need[4], act[4], at;
            for (;; s0 += 256) {              // four sequences to a lane
                int rows[4], all = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) rows[u] = a.n_packed[min(s0 + lane * 4 + u, a.B - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int s = s0 + lane * 4 + u;
                    act[u] = groups_of(rows[u]);
                    need[u] = s < a.B ? wgs_of(s, act[u]) : 0;
                    all += need[u];
                }
                const int sum = running(all);
                const uint64_t past = __builtin_amdgcn_ballot_w64(sum > own);
                if (past != 0) {
                    at = __builtin_ctzll(past);
                    own -= __builtin_amdgcn_readlane(sum, at) - __builtin_amdgcn_readlane(all, at);
                    break;
                }
                own -= __builtin_amdgcn_readlane(sum, 63);
                if (s0 + 256 >= a.B) return;
            }
            b = s0 + at * 4;
            n_act = __builtin_amdgcn_readlane(act[0], at);
#pragma unroll
            for (int u = 0; u < 3; ++u) {     // past the lane's first sequences
                const int n = __builtin_amdgcn_readlane(need[u], at);
                if (b == s0 + at * 4 + u && own >= n) {
                    own -= n;
                    ++b;
                    n_act = __builtin_amdgcn_readlane(act[u + 1], at);
                }
            }
        }
        const int n_wg = n_act * ranges, hl = own / n_wg;
        r_wg = own - hl * n_wg;
        bh = (heads_before(b) + hl) * 8 + xcd;
    }
    if (n_rg > 1) {                           // output rows of the groups without packed rows are zero
        T *z = static_cast<T *>(a.out) + (size_t)bh * a.N * D;
        const int n_wg = ALL ? 1 : n_act * ranges;
        for (int i = n_act * kRows * D + (r_wg * NW * 64 + tid) * 8; i < a.N * D; i += n_wg * NW * 64 * 8)
            *reinterpret_cast<uint4 *>(z + i) = make_uint4(0, 0, 0, 0);
    }
    const int C_b = ctx_len[b], P_b = packed[b];
    const int split = ALL || n_act == 1 ? r_wg : r_wg / n_act;
    int rg = ALL ? 0 : r_wg - split * n_act;
    for (;;) {                                // (ALL: row groups)
    int lane_ = tid & 63, bh_ = bh;
    if constexpr (ALL) asm volatile("" : "+v"(lane_), "+s"(bh_));      // (addresses made anew for every group: kept over the loop they spill)
    const int lane = lane_, bh = bh_, r16 = lane & 15, g = lane >> 4;
    const int row0 = rg * kRows;
    const int Ng = min(kRows, a.N - row0);                      // rows of `out` this group owns
    const int lrow = lane / G::kChunks, lchunk = lane % G::kChunks;

    // ---- Q -> LDS, rows in K's order: copied, or (rotation) through registers, a wave every NW-th (row tile, k-steps t and
    // t + KS/2, which hold a lane's pairs).
    const uintptr_t Qb = reinterpret_cast<uintptr_t>(a.q) + ((size_t)bh * a.N + row0) * RB;
    constexpr int kQPieces = kRows * RB / 1024;
    constexpr int kQFrags = NQ * KS / 2, kQPer = (kQFrags + NW - 1) / NW;
    const int op_rd = r16 * RB + kswz<D>(r16, g) * 16;          // operand order: row r16 of a tile, 16-byte piece 4t + g
    int qpos[kQPer], kpos[2] = {0, 0};                          // kpos: of the first packed-key tile
    uint4 qlo[kQPer], qhi[kQPer];
    if constexpr (ROPE) {
#pragma unroll
        for (int i = 0; i < kQPer; ++i) {
            const int f = min(wave + NW * i, kQFrags - 1), row = min(f / (KS / 2) * 16 + r16, Ng - 1);
            qpos[i] = a.position_ids[(size_t)b * a.N + row0 + row];
            const unsigned char *q = reinterpret_cast<const unsigned char *>(Qb) + row * RB + (4 * (f % (KS / 2)) + g) * 16;
            qlo[i] = ldg16(q);
            qhi[i] = ldg16(q + D);
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) kpos[mt] = a.position_ids[(size_t)b * a.N + min(mt * 16 + r16, a.N - 1)];
    } else {
        for (int p = wave; p < kQPieces; p += NW) {
            const int row = p * G::kRowsPerLoad + lrow;
            dma16(Qb, (uint32_t)(min(row, Ng - 1) * RB + kswz<D>(row, lchunk) * 16), ldsQ + p * 1024);
        }
    }

    const int C = clampi(C_b, 0, a.Cmax);
    const int P_all = clampi(P_b, 0, a.N);
    const int P = clampi(P_all - row0, 0, kRows);
    // a packed row sees no packed key beyond itself (the mask is lower triangular)
    const int tree_end = min(P_all, row0 + kRows);

    // ---- this workgroup's tiles: the tiles of a head are dealt evenly to as few of its `ranges` workgroups as give each
    // at least one tile per wave; the others have nothing to do and nobody waits for them.
    const int nA = (C + 31) >> 5;
    const int nT = P > 0 ? nA + ((tree_end + 31) >> 5) : 0;
    int n_part = 1, tile_begin = 0, tile_end = nT;
    if (ranges > 1) {
        n_part = clampi((nT + NW - 1) / NW, 1, ranges);
        if (split >= n_part) {
            wait_vm<0>();                     // (copies into this workgroup's LDS)
            return;
        }
        const int per = (nT + n_part - 1) / n_part;
        tile_begin = min(split * per, nT);
        tile_end = min(nT, tile_begin + per);
    }
    const int head = bh - b * a.H;
    const int t_first = tile_begin + wave;

    // ---- where a tile's rows are.  Context rows: the cache (paged: the pool); packed rows: k_new, v_new.
    const uintptr_t Kc = reinterpret_cast<uintptr_t>(a.k_cache) + (PAGED ? 0 : (size_t)bh * a.Cmax * RB);
    const uintptr_t Vc = reinterpret_cast<uintptr_t>(a.v_cache) + (PAGED ? 0 : (size_t)bh * a.Cmax * RB);
    const uintptr_t Kn = reinterpret_cast<uintptr_t>(a.k_new) + (size_t)bh * a.N * RB;
    const uintptr_t Vn = reinterpret_cast<uintptr_t>(a.v_new) + (size_t)bh * a.N * RB;
    // Page of a context tile: through the scalar cache as well, one tile ahead of its use.
    auto page_of = [&](int tile) __attribute__((always_inline)) {
        if (!PAGED || tile >= min(nA, tile_end)) return 0;
        const int pg = min(tile * 32 / a.page_size, a.max_pages - 1);
        return clampi(((cint32 *)(uintptr_t)a.block_table)[(size_t)b * a.max_pages + pg], 0, a.n_pages - 1);
    };
    auto tile_off = [&](int tile, int page) __attribute__((always_inline)) -> size_t {   // bytes to the tile's first key
        if (tile >= nA) return (size_t)((uint32_t)(tile - nA) * 32) * RB;
        if (!PAGED) return (size_t)((uint32_t)tile * 32) * RB;
        return (((size_t)page * a.H + head) * a.page_size + (uint32_t)(tile * 32) % (uint32_t)a.page_size) * RB;
    };
    auto tile_keys = [&](int tile) __attribute__((always_inline)) { return min(32, tile >= nA ? tree_end - (tile - nA) * 32 : C - tile * 32); };
    // A tile is copied row by row, the 16-byte pieces of a row in swizzled order (the destination of a lane is fixed, so the
    // order is made by the choice of the source).  Rows past the end of a tile's keys are its last key again; their
    // probabilities are zero.
    auto copy_k = [&](uintptr_t base, int keys) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kLoads; ++s) {
            const int row = s * G::kRowsPerLoad + lrow;
            dma16(base, (uint32_t)(min(row, keys - 1) * RB + kswz<D>(row, lchunk) * 16), ldsK + s * 1024);
        }
    };
    auto copy_v = [&](uintptr_t base, int keys) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kLoads; ++s) {
            const int row = s * G::kRowsPerLoad + lrow;
            dma16(base, (uint32_t)(min(row, keys - 1) * RB + vswz<D>(row, lchunk) * 16), ldsV + s * 1024);
        }
    };
    // Visibility words of the group's rows for one packed-key tile (fetched with every K tile, so that waits can count).
    const uintptr_t mask_b = reinterpret_cast<uintptr_t>(a.mask_bits) + (size_t)b * a.N * a.words * 8;
    const uint32_t mask_row = (uint32_t)min(row0 + lane, a.N - 1) * (uint32_t)a.words * 8;
    auto copy_mask = [&](int tile) __attribute__((always_inline)) { dma4(mask_b + (size_t)clampi(tile - nA, 0, 2 * a.words - 1) * 4, mask_row, ldsMask); };

    // ---- the first tile.  A wave that turns rows of Q asks for its tile behind that (the wait for the angles would else be one
    // for K and V), the other waves' tiles keep the memory busy meanwhile.
    const int nqt = (P + 15) >> 4;
    int page = page_of(t_first);
    const bool some = t_first < tile_end;
    if constexpr (ROPE) {
#pragma unroll
        for (int i = 0; i < kQPer; ++i) {
            const int f = wave + NW * i, t = f % (KS / 2);
            if (f < kQFrags && f / (KS / 2) < nqt) {
                const size_t o = (size_t)clampi(qpos[i], 0, a.max_pos - 1) * (D / 2) + (4 * t + g) * 8;
                float cs[8], sn[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) { cs[e] = a.cos_tab[o + e]; sn[e] = a.sin_tab[o + e]; }
                unsigned char *q = sQ + f / (KS / 2) * 16 * RB;
                *reinterpret_cast<uint4 *>(q + (op_rd ^ (4 * t * 16))) = rope8<T>(qlo[i], qhi[i], cs, sn, true);
                *reinterpret_cast<uint4 *>(q + (op_rd ^ (4 * (t + KS / 2) * 16))) = rope8<T>(qhi[i], qlo[i], cs, sn, false);
            }
        }
    }
    if (some) {
        const size_t off = tile_off(t_first, page);
        copy_mask(t_first);
        copy_k((t_first >= nA ? Kn : Kc) + off, tile_keys(t_first));
        copy_v((t_first >= nA ? Vn : Vc) + off, tile_keys(t_first));
    }
    page = page_of(t_first + NW);
    if constexpr (!ROPE) {
        if (some) wait_vm<2 * kLoads + 1>();  // this wave's part of Q is there
        else wait_vm<0>();
    }
    RD_TR(9);
    rd_lds_barrier();                            // Q visible to all waves
    RD_TR(1);

    const float c_abs = fabsf(a.scale_log2e);
    const bool c_neg = a.scale_log2e < 0.f;
    auto op = [&](const unsigned char *tile, int mt, int t) __attribute__((always_inline)) {
        return *reinterpret_cast<const vec8 *>(tile + mt * 16 * RB + (op_rd ^ ((4 * t & (G::kChunks - 1)) * 16)));
    };
    const unsigned char *myK = sK + wave * G::kTileBytes;
    const int v_row = 4 * g + (r16 >> 2), v_rd = v_row * RB + vswz<D>(v_row, (r16 & 3) >> 1) * 16 + (r16 & 1) * 8;
    auto v_frag = [&](int tile, int dt) __attribute__((always_inline)) {          // V^T of wave `tile`'s tile, d-tile dt, as an A operand
        const unsigned char *vt = sV + tile * G::kTileBytes + (v_rd ^ ((dt & (G::kChunks / 2 - 1)) * 32));
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)vt);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(vt + 16 * RB));
        return __builtin_bit_cast(vec8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    T *outp = static_cast<T *>(a.out) + ((size_t)bh * a.N + row0) * D;
    auto put = [&](int qt, int dt, f32x4 o, float l) __attribute__((always_inline)) {
        const int row = qt * 16 + r16;
        if (row < Ng) {
            const bool keep = row < P;                          // rows beyond the packed count are zero
            const float inv = keep ? 1.0f / l : 0.f;
            f32x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = keep ? o[e] * inv : 0.f;
                asm volatile("" : "+v"(v));                     // an fp32 product, then one rounding, in every instance
                y[e] = v;
            }
            store_out4(outp + (size_t)row * D + dt * 16 + 4 * g, y[0], y[1], y[2], y[3]);
        }
    };

    // Instantiated for all row tiles and for the lower half (a padded row tile costs as much as a real one).
    auto walk = [&](auto nqa_tag) __attribute__((always_inline)) {
        constexpr int NQA = decltype(nqa_tag)::value;
        constexpr int kRoundsA = (NQA + 1) / 2;
        // The rotated rows of a packed-key tile also go to a.k_rot (what a cache stores).
        auto store_rot = [&](int tile, const vec8 (&kreg)[2][KS]) __attribute__((always_inline)) {
            if (a.k_rot == nullptr) return;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const int key = (tile - nA) * 32 + mt * 16 + r16;
                if (key < tree_end) {
                    unsigned char *kr = static_cast<unsigned char *>(a.k_rot) + ((size_t)bh * a.N + key) * RB + g * 16;
#pragma unroll
                    for (int t = 0; t < KS; ++t) *reinterpret_cast<vec8 *>(kr + 64 * t) = kreg[mt][t];
                }
            }
        };
        // Scores of one tile, keys x rows, from the K tile and visibility words in LDS; `prefetch` runs as soon as those are read;
        // `only`: it is the wave's only tile.
        // In log2 units they are the result times the factor returned.
        auto scores = [&](int tile, vec8 (&kreg)[2][KS], f32x4 (&sacc)[2][NQA], auto only, auto prefetch) __attribute__((always_inline)) {
            const bool tree = tile >= nA;
            uint32_t vis[NQA];
            // Packed keys are rotated here.  A lane's angles of half a tile's k-step:
            constexpr bool kEarly = ROPE && decltype(only)::value;
            typedef float angles[2][8];
            size_t at[2] = {0, 0};
            auto load_angles = [&](int mt, int t, angles &x) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) { x[0][e] = a.cos_tab[at[mt] + t * 32 + e]; x[1][e] = a.sin_tab[at[mt] + t * 32 + e]; }
            };
            angles early[kEarly ? 2 : 1][kEarly ? KS / 2 : 1];
            if constexpr (ROPE) {
                if (tree) {
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt) {
                        int pos = kpos[mt];
                        if (tile != nA) pos = a.position_ids[(size_t)b * a.N + min((tile - nA) * 32 + mt * 16 + r16, a.N - 1)];
                        at[mt] = (size_t)clampi(pos, 0, a.max_pos - 1) * (D / 2) + g * 8;
#pragma unroll
                        for (int t = 0; t < KS / 2; ++t)
                            if constexpr (kEarly) load_angles(mt, t, early[mt][t]);      // (in the loop the registers are not there)
                    }
                }
            }
            wait_vm<kLoads>();                // K and mask of this tile (its V is younger)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int t = 0; t < KS; ++t) kreg[mt][t] = op(myK, mt, t);
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) vis[qt] = *reinterpret_cast<const uint32_t *>(sMask + wave * 256 + (qt * 16 + r16) * 4);
            // Q's operands are read kAhead k-steps before they are multiplied: read when needed, a lone wave waits for LDS at each
            // of them.  LDS answers in order: with theirs outstanding K's reads are done.
            // (With three row tiles and the angles the registers for two are not there, and at D = 64 four waves of more than 168
            // leave two workgroups to a compute unit instead of three: us when needed / one ahead, H=32, B=16, 70 x 5 tokens, C=300
            // 44.8 / 53.2, B=64, 16 x 5, C=200 39.3 / 44.9.  Eight waves are alone on it either way: H=32, C=2000 10.3 / 9.9.)
            constexpr int kAhead = ROPE && NQA == 3 ? (D == 64 && NW == 4 ? 0 : 1) : 2;
            vec8 bq[KS][NQA];
            auto read_q = [&](int t) __attribute__((always_inline)) {
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) bq[t][qt] = op(sQ, qt, t);
            };
            asm volatile("" : : : "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < kAhead; ++t) read_q(t);
            wait_lds<kAhead * NQA>();
            prefetch();
            if constexpr (ROPE) {
                if (tree) {
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
                        for (int t = 0; t < KS / 2; ++t) {
                            angles late;
                            if constexpr (!kEarly) load_angles(mt, t, late);
                            const angles &x = kEarly ? early[kEarly ? mt : 0][kEarly ? t : 0] : late;
                            const uint4 lo = __builtin_bit_cast(uint4, kreg[mt][t]), hi = __builtin_bit_cast(uint4, kreg[mt][t + KS / 2]);
                            kreg[mt][t] = __builtin_bit_cast(vec8, rope8<T>(lo, hi, x[0], x[1], true));
                            kreg[mt][t + KS / 2] = __builtin_bit_cast(vec8, rope8<T>(hi, lo, x[0], x[1], false));
                        }
                    }
                    if constexpr (!kEarly) store_rot(tile, kreg);
                }
            }
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) sacc[0][qt] = sacc[1][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                if (t + kAhead < KS) read_q(t + kAhead);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) {
                    sacc[0][qt] = Elem<T>::mfma(kreg[0][t], bq[t][qt], sacc[0][qt]);
                    sacc[1][qt] = Elem<T>::mfma(kreg[1][t], bq[t][qt], sacc[1][qt]);
                }
            }

            // softmax in log2 units.  An interior context tile keeps the raw scores (the scale is folded into
            // the exponent); a tile with masked or missing keys is scaled here and its dead entries set to -inf.
            // Element (mt, i) of a lane's scores is key 16*mt + 4g + i.
            const int rem = tile_keys(tile);
            const bool plain = !tree && rem >= 32 && !c_neg;
            if (!plain) {
                const uint32_t tail = rem >= 32 ? 0xffffffffu : ((1u << rem) - 1u);
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) {
                    const uint32_t bits = ((tree ? vis[qt] : 0xffffffffu) & tail) >> (4 * g);
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            sacc[mt][qt][i] = ((bits >> (16 * mt + i)) & 1u) ? sacc[mt][qt][i] * a.scale_log2e : -INFINITY;
                }
            }
            return plain ? c_abs : 1.0f;
        };
        auto tile_max = [&](const f32x4 (&sacc)[2][NQA], int qt) __attribute__((always_inline)) {
            return quad_max(fmaxf(fmaxf(fmaxf(sacc[0][qt][0], sacc[0][qt][1]), fmaxf(sacc[0][qt][2], sacc[0][qt][3])),
                                  fmaxf(fmaxf(sacc[1][qt][0], sacc[1][qt][1]), fmaxf(sacc[1][qt][2], sacc[1][qt][3]))));
        };
        auto weights = [&](const f32x4 (&sacc)[2][NQA], int qt, float c_fold, float m_safe) __attribute__((always_inline)) {
            vec8 pb;
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) pb[4 * mt + i] = (T)__builtin_amdgcn_exp2f(__builtin_fmaf(sacc[mt][qt][i], c_fold, -m_safe));
            return pb;
        };
        // Sums of the rows' probabilities as they were rounded (what is added up of V has just these weights), by a matrix
        // instruction with ones in V's place: the same in all elements.
        vec8 ones;
#pragma unroll
        for (int i = 0; i < 8; ++i) ones[i] = (T)1.f;
        // The waves' statistics of a row, by all lanes.
        auto stats = [&](const float *table, int qt, float (&x)[NW]) __attribute__((always_inline)) {
#pragma unroll
            for (int w = 0; w < NW; w += 4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(table + (qt * 16 + r16) * kStat + w);
                x[w] = v[0]; x[w + 1] = v[1]; x[w + 2] = v[2]; x[w + 3] = v[3];
            }
        };
        float m_run[NQA], l_run[NQA];         // in the end: reference and sum of every row
        f32x4 own[kRoundsA][kOwn];            // ... and this wave's fragments of the result: number f of round r is row tile
                                              // 2r + f / DT, d-tile f % DT
        auto row_tile = [&](int r, int j) __attribute__((always_inline)) { return 2 * r + (j * NW + wave) / DT; };
        auto d_tile = [&](int j) __attribute__((always_inline)) { return (j * NW + wave) % DT; };
        auto pick = [&](const float (&x)[NQA], int r, int j) __attribute__((always_inline)) {     // x[row tile]
            const float lo = x[2 * r], hi = x[2 * r + 1 < NQA ? 2 * r + 1 : 2 * r];
            return (j * NW + wave) / DT ? hi : lo;
        };
        if (tile_end - tile_begin <= NW) {
            // At most one tile per wave: every wave adds up its own fragments over all the tiles, whose probabilities and V are in
            // LDS.  A tile's probabilities are taken against its own maximum and its product is scaled: against one reference for
            // all of them, 0.1 us less at H=32, C=1024, those of a tile far below it are subnormal in fp16, and no tile but one
            // has its largest exact (bf16, 40 rows, C=1024: relative error 2.17e-3 instead of 2.02e-3).
            vec8 kreg[2][KS];
            f32x4 sacc[2][NQA];
            float c_fold = 1.f;
            // Tiles that are added up below.  Waves past them write nothing: zeros from every idle wave are half a tile's time
            // (us with / without, D = 128: B=47, H=26, C=46, 6 tokens 10.2 / 9.5; B=55, H=12, C=33, 16 tokens 6.7 / 6.2).
            const int n_tiles = tile_end - tile_begin, n_sum = n_tiles <= NW / 2 ? NW / 2 : n_tiles <= NW / 2 + NW / 4 ? NW / 2 + NW / 4 : NW;
            if (some) {
                c_fold = scores(t_first, kreg, sacc, std::true_type{}, []() {});
            } else if (wave < n_sum) {        // no tile: zeros for the sum over the tiles below
#pragma unroll
                for (int s = 0; s < kLoads; ++s) *reinterpret_cast<uint4 *>(sV + wave * G::kTileBytes + s * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) *reinterpret_cast<uint4 *>(sK + wave * G::kTileBytes + (qt * 64 + lane) * 16) = make_uint4(0, 0, 0, 0);
            }
            RD_TR(2);
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                float mx = -INFINITY;
                f32x4 sum = {0.f, 0.f, 0.f, 0.f};
                if (some) {
                    mx = tile_max(sacc, qt) * c_fold;
                    const vec8 pb = weights(sacc, qt, c_fold, mx == -INFINITY ? 0.f : mx);
                    *reinterpret_cast<vec8 *>(sK + wave * G::kTileBytes + (qt * 64 + lane) * 16) = pb;
                    sum = Elem<T>::mfma(ones, pb, sum);
                }
                if (g == 0) {
                    sM[(qt * 16 + r16) * kStat + wave] = mx;
                    sL[(qt * 16 + r16) * kStat + wave] = sum[0];
                }
            }
            wait_vm<0>();                     // this wave's V tile
            rd_lds_barrier();                    // probabilities, statistics and V of all waves visible
            RD_TR(8);
            float fac[NQA][NW];               // 2^(reference of a tile - reference of the row)
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                float y[NW];
                stats(sM, qt, fac[qt]);
                stats(sL, qt, y);
                float m = fac[qt][0];
#pragma unroll
                for (int w = 1; w < NW; ++w) m = fmaxf(m, fac[qt][w]);
                m_run[qt] = m;
                l_run[qt] = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    fac[qt][w] = __builtin_amdgcn_exp2f(fac[qt][w] - (m == -INFINITY ? 0.f : m));
                    l_run[qt] += fac[qt][w] * y[w];
                }
            }
#pragma unroll
            for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
                for (int j = 0; j < kOwn; ++j) own[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            constexpr int kD = DT >= NW ? DT / NW : 1;          // d-tiles of a wave's fragments: those of j = 0 .. kD-1
            // NW / 2 tiles (with more than one range a workgroup has more than that) and the rest by quarters, without branches in
            // between: the reads run ahead.  (The rest at once adds up to three tiles of zeros: us with / without, B=3, H=8, C=94, 96
            // tokens 6.95 / 6.60, B=8, H=32, C=122, 16 tokens 4.32 / 4.17.)
            auto add_tiles = [&](auto first, auto count) __attribute__((always_inline)) {
#pragma unroll
                for (int kt = decltype(first)::value; kt < decltype(first)::value + decltype(count)::value; ++kt) {
                    float f[NQA];
#pragma unroll
                    for (int qt = 0; qt < NQA; ++qt) f[qt] = fac[qt][kt];
                    vec8 vf[kD];
#pragma unroll
                    for (int j = 0; j < kD; ++j) vf[j] = v_frag(kt, d_tile(j));
#pragma unroll
                    for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
                        for (int j = 0; j < kOwn; ++j) {
                            if (DT >= NW && 2 * r + j / kD >= NQA) continue;
                            const vec8 pb = *reinterpret_cast<const vec8 *>(sK + kt * G::kTileBytes + (min(row_tile(r, j), NQA - 1) * 64 + lane) * 16);
                            own[r][j] += pick(f, r, j) * Elem<T>::mfma(vf[j % kD], pb, f32x4{0.f, 0.f, 0.f, 0.f});
                        }
                }
            };
            using half = std::integral_constant<int, NW / 2>;
            using three = std::integral_constant<int, NW / 2 + NW / 4>;
            using quarter = std::integral_constant<int, NW / 4>;
            add_tiles(std::integral_constant<int, 0>{}, half{});
            if (n_sum > half::value) {
                add_tiles(half{}, quarter{});
                if (n_sum > three::value) add_tiles(three{}, quarter{});
            }
            if constexpr (ROPE) {             // (not before V is waited for: that would be a wait for these stores)
                if (some && t_first >= nA) store_rot(t_first, kreg);
            }
            RD_TR(3);
        } else {
        float m_ref[NQA];                     // exponents' reference of every row
        f32x4 l_own[NQA], oacc[NQA][DT];      // the sums, the output
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) {
            m_ref[qt] = -INFINITY;
            l_own[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int tile = t_first; tile < tile_end; tile += NW) {
            const bool more = tile + NW < tile_end, tree = tile >= nA;
            const int next = tile + NW;
            const size_t off_next = tile_off(next, page);
            const int keys_next = tile_keys(next);
            vec8 kreg[2][KS];
            f32x4 sacc[2][NQA];
            const float c_fold = scores(tile, kreg, sacc, std::false_type{}, [&]() __attribute__((always_inline)) {
                if (more) {
                    copy_mask(next);
                    copy_k((next >= nA ? Kn : Kc) + off_next, keys_next);
                }
                page = page_of(next + NW);
            });
            if (more) wait_vm<kLoads + 1>();  // V of this tile (the next K and mask are younger)
            else wait_vm<0>();
            vec8 vreg[DT];                    // read while the exponents are taken
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) vreg[dt] = v_frag(wave, dt);
            // Reference of the exponents: the running one, or this tile's maximum in rows where it lies more than
            // 2^kSlack above that.  Rows seldom move once the first tile is in, and while none does the products add
            // up without a factor.
            float ref[NQA];
            bool moved = false;
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                const float mx = tile_max(sacc, qt) * c_fold;
                const bool up = mx > m_ref[qt] + kSlack;
                moved |= up;
                ref[qt] = up ? mx : m_ref[qt];
            }
            if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) {
                    const float alpha = __builtin_amdgcn_exp2f(m_ref[qt] - (ref[qt] == -INFINITY ? 0.f : ref[qt]));
                    l_own[qt] *= alpha;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] *= alpha;
                    m_ref[qt] = ref[qt];
                }
            }
            vec8 pb[NQA];
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                pb[qt] = weights(sacc, qt, c_fold, m_ref[qt] == -INFINITY ? 0.f : m_ref[qt]);
                l_own[qt] = Elem<T>::mfma(ones, pb[qt], l_own[qt]);
            }
            wait_lds();
            if (more) copy_v((next >= nA ? Vn : Vc) + off_next, keys_next);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) oacc[qt][dt] = Elem<T>::mfma(vreg[dt], pb[qt], oacc[qt][dt]);
        }
        RD_TR(3);

        // ---- the waves' states meet in LDS
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) {
            if (g == 0) {
                sM[(qt * 16 + r16) * kStat + wave] = m_ref[qt];
                sL[(qt * 16 + r16) * kStat + wave] = l_own[qt][0];
            }
        }
        rd_lds_barrier();                        // states of all waves visible, all tiles read
#pragma unroll
        for (int qt = 0; qt < NQA; ++qt) {
            float x[NW], y[NW];
            stats(sM, qt, x);
            stats(sL, qt, y);
            float m = x[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) m = fmaxf(m, x[w]);
            const float m_safe = m == -INFINITY ? 0.f : m;
            m_run[qt] = m;
            l_run[qt] = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) l_run[qt] += __builtin_amdgcn_exp2f(x[w] - m_safe) * y[w];
            const float f = __builtin_amdgcn_exp2f(m_ref[qt] - m_safe);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[qt][dt] *= f;
        }
#pragma unroll
        for (int r = 0; r < kRoundsA; ++r) {
            if (r > 0) rd_lds_barrier();
#pragma unroll
            for (int ql = 0; ql < 2; ++ql)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    if (2 * r + ql < NQA) *reinterpret_cast<f32x4 *>(sK + ((wave * 2 * DT + ql * DT + dt) * 64 + lane) * 16) = oacc[2 * r + ql < NQA ? 2 * r + ql : 0][dt];
            rd_lds_barrier();
#pragma unroll
            for (int j = 0; j < kOwn; ++j) {
                const int f = j * NW + wave;
                own[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (2 * r + 1 < NQA || f < DT)
#pragma unroll
                    for (int w = 0; w < NW; ++w) own[r][j] += *reinterpret_cast<const f32x4 *>(sK + ((w * 2 * DT + f) * 64 + lane) * 16);
            }
        }
        }
        if (n_part == 1) {                    // the group's only workgroup
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
#pragma unroll
                for (int j = 0; j < kOwn; ++j)
                    if (row_tile(r, j) < NQ) put(row_tile(r, j), d_tile(j), own[r < kRoundsA ? r : 0][j], r < kRoundsA ? pick(l_run, r < kRoundsA ? r : 0, j) : 1.f);
            RD_TR(6);
            return;
        }

        // ---- partial state -> workspace; the last workgroup of this head (and row group) merges.
        // Layout of one partial: (m, l) per row, then the fragments [row tile][d-tile][64 lanes][4], so that
        // every wave store and load covers 1 KB.
        const size_t unit = (size_t)bh * n_rg + rg;
        float *part = a.partials + ((size_t)bh * a.S + split * n_act + rg) * kPF;
        auto frag = [&](int r, int j) __attribute__((always_inline)) { return 2 * kRows + ((row_tile(r, j) * DT + d_tile(j)) * 64 + lane) * 4; };
#pragma unroll
        for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
            for (int j = 0; j < kOwn; ++j) {
                const int qt = row_tile(r, j);
                if (qt < NQA && qt * 16 + r16 < P) {
                    if (d_tile(j) == 0 && g == 0) st_dev2(part + 2 * (qt * 16 + r16), pick(m_run, r, j), pick(l_run, r, j));
                    st_dev4(part + frag(r, j), own[r][j][0], own[r][j][1], own[r][j][2], own[r][j][3]);
                }
            }
        RD_TR(4);
        const int last = arrive_is_last(a.counters + unit, (uint32_t)n_part);
        RD_TR(5);
        if (last == kNotLast) return;
        // All loads of a chunk of partials are in flight together; no branch stands before one (partials past the end
        // are the last one again with weight zero, rows that hold nothing are never written), so the chunk follows their number.
        const float *hp = a.partials + ((size_t)bh * a.S + rg) * kPF;
        auto merge = [&](auto clean, auto chunk) __attribute__((always_inline)) {
            constexpr int kChunk = decltype(chunk)::value;
            f32x4 acc[kRoundsA][kOwn];
            float M[NQA], den[NQA];
#pragma unroll
            for (int qt = 0; qt < NQA; ++qt) {
                M[qt] = -INFINITY;
                den[qt] = 0.f;
            }
#pragma unroll
            for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
                for (int j = 0; j < kOwn; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int s0 = 0; s0 < n_part; s0 += kChunk) {
                float2 ml[NQA][kChunk];
                f32x4 fr[kRoundsA][kOwn][kChunk];
#pragma unroll
                for (int c = 0; c < kChunk; ++c) {
                    const float *ps = hp + (size_t)min(s0 + c, n_part - 1) * n_act * kPF;
#pragma unroll
                    for (int qt = 0; qt < NQA; ++qt) {
                        const float *pm = ps + qt * 32 + 2u * (unsigned)r16;
                        ml[qt][c] = decltype(clean)::value ? *reinterpret_cast<const float2 *>(pm) : ld_dev2(pm);
                    }
#pragma unroll
                    for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
                        for (int j = 0; j < kOwn; ++j) {
                            if (DT >= NW && 2 * r + j * NW / DT >= NQA) continue;
                            const float *pf = ps + 2 * kRows + (min(row_tile(r, j), NQA - 1) * DT + d_tile(j)) * 256 + 4u * (unsigned)lane;
                            if (decltype(clean)::value) {
                                fr[r][j][c] = *reinterpret_cast<const f32x4 *>(pf);
                            } else {
                                const float2 lo = ld_dev2(pf), hi = ld_dev2(pf + 2);
                                fr[r][j][c] = f32x4{lo.x, lo.y, hi.x, hi.y};
                            }
                        }
                }
                float w[NQA][kChunk], resc[NQA];
#pragma unroll
                for (int qt = 0; qt < NQA; ++qt) {
                    float Mn = M[qt];
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) {
                        ml[qt][c].x = s0 + c < n_part ? ml[qt][c].x : -INFINITY;
                        Mn = fmaxf(Mn, ml[qt][c].x);
                    }
                    const float Ms = Mn == -INFINITY ? 0.f : Mn;
                    resc[qt] = __builtin_amdgcn_exp2f(M[qt] - Ms);
                    den[qt] *= resc[qt];
#pragma unroll
                    for (int c = 0; c < kChunk; ++c) {
                        w[qt][c] = __builtin_amdgcn_exp2f(ml[qt][c].x - Ms);
                        den[qt] += w[qt][c] * ml[qt][c].y;
                    }
                    M[qt] = Mn;
                }
#pragma unroll
                for (int r = 0; r < kRoundsA; ++r)
#pragma unroll
                    for (int j = 0; j < kOwn; ++j) {
                        if (DT >= NW && 2 * r + j * NW / DT >= NQA) continue;
                        acc[r][j] *= pick(resc, r, j);
#pragma unroll
                        for (int c = 0; c < kChunk; ++c) {
                            float wc[NQA];
#pragma unroll
                            for (int qt = 0; qt < NQA; ++qt) wc[qt] = w[qt][c];
                            acc[r][j] += pick(wc, r, j) * fr[r][j][c];
                        }
                    }
            }
            RD_TR(7);
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
#pragma unroll
                for (int j = 0; j < kOwn; ++j)
                    if (row_tile(r, j) < NQ) put(row_tile(r, j), d_tile(j), acc[r < kRoundsA ? r : 0][j], r < kRoundsA ? pick(den, r < kRoundsA ? r : 0, j) : 1.f);
        };
        using std::integral_constant;
        // Partials of several XCDs are not seen where workgroups are dealt to them in turn; their reads, 8 bytes each past the L2,
        // take chunks of two (us by 2 / 4: H=32, C=1024, 8 x 5 tokens 12.1 / 13.3, C=2048, 16 x 5 22.5 / 23.4; H=8, C=6000, 3 x 5,
        // many small partials, 14.3 / 13.6).
        if (last != kLastClean) merge(std::false_type{}, integral_constant<int, 2>{});
        else if (n_part <= 4 || kRoundsA * kOwn * 8 > 24) merge(std::true_type{}, integral_constant<int, 4>{});
        else if (n_part <= 6) merge(std::true_type{}, integral_constant<int, 6>{});
        else merge(std::true_type{}, integral_constant<int, 8>{});
        if (tid == 0) a.counters[unit] = 0;   // leave the workspace ready for the next call
        RD_TR(6);
    };
    constexpr int kHalf = (NQ + 1) / 2;
    if (NQ > 1 && nqt <= kHalf) walk(std::integral_constant<int, kHalf>{});
    else walk(std::integral_constant<int, NQ>{});
    if (!ALL || ++rg >= n_act) return;
    rd_lds_barrier();                            // all waves have read what the next group's copies overwrite
    }
}

template <int D, int NQ, int NW>
static constexpr size_t mfma_smem_bytes()
{
    return (size_t)2 * NW * Geo<D>::kTileBytes + (size_t)NQ * 16 * Geo<D>::kRowBytes + NW * 256 + (size_t)2 * NQ * 16 * stat_stride(NW) * sizeof(float);
}

template <typename T, int D, int NQ, int NW, bool PAGED, bool ROPE, bool ALL = false>
static int launch_mfma(const AttnArgs &a, hipStream_t stream)
{
    constexpr size_t smem = mfma_smem_bytes<D, NQ, NW>();
    static_assert((smem + 256) * (8 / NW) <= 160 * 1024, "LDS of a compute unit: one workgroup of eight waves, two of four");
    static std::atomic<unsigned long long> configured{0};
    const int st = ensure_dynamic_lds(reinterpret_cast<const void *>(&rd_tree_attn_mfma_kernel<T, D, NQ, NW, PAGED, ROPE, ALL>), smem, configured);
    if (st != RD_OK) return st;
    const size_t wgs = ((size_t)a.B * a.H + 7) / 8 * 8 * a.S;
    if (wgs > 0x7fffffffull) return RD_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((rd_tree_attn_mfma_kernel<T, D, NQ, NW, PAGED, ROPE, ALL>), dim3((unsigned)wgs), dim3(NW * 64), smem, stream, a);
    return rd_check_launch();
}

template <typename T, int D, int NW, bool PAGED, bool ROPE>
static int dispatch_nq(const AttnArgs &a, int rg_tiles, hipStream_t stream)
{
    if constexpr (NW == 4) {
        if (a.n_rg > 1 && a.S == 1) {
            if (rg_tiles == 2) return launch_mfma<T, D, 2, NW, PAGED, ROPE, true>(a, stream);
            if (rg_tiles == 3) return launch_mfma<T, D, 3, NW, PAGED, ROPE, true>(a, stream);
            return RD_ERR_UNSUPPORTED;
        }
    }
    switch (rg_tiles) {
    case 1: return launch_mfma<T, D, 1, NW, PAGED, ROPE>(a, stream);
    case 2: return launch_mfma<T, D, 2, NW, PAGED, ROPE>(a, stream);
    case 3: return launch_mfma<T, D, 3, NW, PAGED, ROPE>(a, stream);
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
