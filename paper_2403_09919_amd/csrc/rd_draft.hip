// rd_draft: the draft model and its beam search (Sec. 3.1, 3.2) for gfx950.
//
// Per drafted position the work is two kinds of launches on the caller's stream:
//   * skinny linear layers  Y[M,N] = X[M,K] W[N,K]^T  with M = B*W rows (one per live candidate)
//     and bf16 weights streamed once from HBM: the layers are bound by that stream (the LM-head
//     alone is V x 2Dm), so a workgroup owns 16 to 64 output columns, its waves split K, weights
//     go from memory straight into the A operand of v_mfma_f32_16x16x32_bf16 (lane = one output
//     column x 8 consecutive k), the activations (a few hundred KB, L2 resident) into the B
//     operand, and the partial sums meet in LDS.  Bias, SiLU, skip connection and the bf16
//     copy that the next layer reads are fused into the epilogue.  Large layers of up to 8 rows take both
//     operands through rings in LDS (rd_stream_kernel).  Layers of many rows, and large ones
//     from 9 rows on, run on a kernel of 256-column workgroups with K split over them, fed through LDS
//     (rd_gemm_kernel), and a second one adds the partial tiles (launch_linear has the rules);
//   * selection: per chunk of 4096 logits and row, the pieces of the log-sum-exp and the W best tokens;
//     per row, its log-sum-exp and the W best tokens of its chunks as cumulative scores; per sequence,
//     the best W of the (candidate, token) pairs by cumulative log probability, ties to the smaller
//     candidate, then the smaller token.  Up to 28 candidates by counting, the last two in one launch
//     where a sequence's lists have a thread each; beyond that three launches, merges of sorted lists
//     (W <= 128; beyond 64 candidates a lane of the last merge holds two lists).
// The RNN update reads its two inputs in place: the parent's state through a row map and the
// chosen token's embedding straight from the table, so no gather pass exists.
//
// Precision contract: weights, embeddings and h are bf16; every linear layer reads its input
// rounded to bf16 and accumulates in fp32; bias, activation, skip connection, log-softmax and
// scores are fp32.
#include "rd_internal.h"
#include <math.h>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

// The 16-bit storage type of the model (bf16 or fp16): eight-element vector and its MFMA.
template <typename T> struct Elem16;
template <> struct Elem16<__bf16> {
    typedef bf16x8 vec8;
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Elem16<_Float16> {
    typedef f16x8 vec8;
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

constexpr int kMaxRows = 512;          // B*W
constexpr int kMaxBeam = 128;          // W
constexpr int kNarrowBeam = 64;        // up to here the selection kernels keep their lists in static LDS, one candidate per lane
// Up to here candidates are ranked by counting, us per call so and by merges (three sequences, hidden size 512, 32000 tokens):
// 16 candidates 171 / 227, 24 230 / 286, 28 253 / 303; 32, for whom the lower bound of 32 groups is too low, 390 / 317.
constexpr int kFewBeam = 28;
constexpr int kSelThreads = 256;       // row pass and beam step: four waves bring the lists into LDS, the first one merges
constexpr int kMaxVocab = 262144;      // 64 chunks of 4096 logits: one lane per chunk in the row pass
constexpr int kSplitMaxWgs = 256;      // workgroups of a launch whose K is split over workgroups
constexpr int kGemmCols = 16;          // its column tiles per workgroup

enum { EPI_HEAD = 0, EPI_RNN = 1, EPI_MLP = 2 };

template <typename T>
struct LinArgs {
    // Y = X1 W1^T (+ X2 W2^T) + bias;  W row-major [N][K]; X rows found through row maps
    const T *w1, *w2;
    const T *x1, *x2;             // row r of X1 is x1 + map1[r]*ldx1 (map NULL: r itself)
    const int32_t *map1, *map2;
    int ldx1, ldx2, K1, K2;            // K2 = 0: single product
    int tiled;                         // weights in the operand-tiled layout of rd_draft_pack_weights
    const float *bias;                 // [N] or NULL
    int M, N;
    int m0;                            // first logical row of this launch (a launch covers rows m0 .. m0+M-1)
    int mstride;                       // logical row m of X (without a map), Y and res is physical row m*mstride
    // epilogue
    float *y_f32;                      // HEAD: logits [M][ldy];  RNN/MLP: activations fp32 [M][ldy]
    T *y_bf;                           // RNN/MLP: the same rounded to the storage type [M][ldy]
    T *s_bf;                           // RNN: next state [M][N]
    const float *res;                  // MLP: skip input fp32 [M][ldy]
    int ldy;
    // rd_gemm_kernel: K split over workgroups
    int ksplit;                        // splits per column group
    int cols;                          // rd_gemm_kernel: column tiles of a workgroup
    float *kpart;                      // partial tiles [group][split][tile][64 lanes] x 4 floats
};

__device__ __forceinline__ float silu(float x) { return x / (1.0f + __expf(-x)); }

// One output tile (16 rows x 16 columns) leaves the kernel: bias, activation, skip connection and the
// bf16 copy that the next layer reads.  Accumulator layout: element i of lane (r16, g) is output
// column n_tile + 4g + i of logical row m_tile + r16.
struct EpilogueIn { f32x4 bias, res; };
template <typename T, int EPI>
__device__ __forceinline__ EpilogueIn linear_epilogue_in(const LinArgs<T> &a, int m_tile, int n_tile, int r16, int g)
{
    EpilogueIn in = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    if (EPI == EPI_HEAD) return in;
    const int n0 = min(n_tile + 4 * g, a.N - 4);                // (N is a multiple of 64 here)
    if (a.bias) {
        const rd::f4_any bias = *reinterpret_cast<const rd::f4_any *>(a.bias + n0);
        in.bias = f32x4{bias[0], bias[1], bias[2], bias[3]};
    }
    if (EPI == EPI_MLP) in.res = *reinterpret_cast<const f32x4 *>(a.res + (size_t)(a.m0 + min(m_tile + r16, a.M - 1)) * a.mstride * a.ldy + n0);
    return in;
}
template <typename T, int EPI>
__device__ __forceinline__ void linear_epilogue(const LinArgs<T> &a, f32x4 v, int m_tile, int n_tile, int r16, int g, const EpilogueIn &in)
{
    const int m = m_tile + r16;
    if (m >= a.M) return;
    const size_t prow = (size_t)(a.m0 + m) * a.mstride;         // physical row of the activation buffers
    const int n0 = n_tile + 4 * g;
    if (EPI == EPI_HEAD) {
        float *y = a.y_f32 + prow * a.ldy + n0;
        if (a.bias == nullptr && n0 + 4 <= a.N) {               // (the logit rows start at any multiple of 4 bytes)
            *reinterpret_cast<rd::f4_any *>(y) = rd::f4_any{v[0], v[1], v[2], v[3]};
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (n0 + i < a.N) y[i] = v[i] + (a.bias ? a.bias[n0 + i] : 0.f);
        return;
    }
    if (n0 >= a.N) return;                                      // (N is a multiple of 64 here)
    typedef __attribute__((ext_vector_type(4))) T vec4;
    const size_t o = prow * a.ldy + n0;
    f32x4 y;
    vec4 yb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float t = silu(v[i] + in.bias[i]);
        if (EPI == EPI_MLP) t += in.res[i];
        y[i] = t;
        yb[i] = (T)t;
    }
    *reinterpret_cast<f32x4 *>(a.y_f32 + o) = y;
    *reinterpret_cast<vec4 *>(a.y_bf + o) = yb;
    if (EPI == EPI_RNN) *reinterpret_cast<vec4 *>(a.s_bf + prow * a.N + n0) = yb;
}
template <typename T, int EPI>
__device__ __forceinline__ void linear_epilogue(const LinArgs<T> &a, f32x4 v, int m_tile, int n_tile, int r16, int g)
{
    if (m_tile + r16 >= a.M || (EPI != EPI_HEAD && n_tile + 4 * g >= a.N)) return;      // (nothing is fetched for tiles past the end)
    linear_epilogue<T, EPI>(a, v, m_tile, n_tile, r16, g, linear_epilogue_in<T, EPI>(a, m_tile, n_tile, r16, g));
}

// A workgroup owns NT*16 output columns for all M = MT*16 rows; its NWV waves split K.  The host
// picks NT so that the activations, which every workgroup re-reads through the caches, do not
// outweigh the weights it streams (their ratio is MT : NT) while the launch still covers the chip,
// and NWV so that the launch has enough waves in flight to keep the HBM stream busy; every wave's
// share of K is a whole number of 32-wide steps inside one of the two products.
template <typename T, int MT, int NT, int NWV, int EPI, bool TILED>
__global__ __launch_bounds__(NWV * 64) void rd_linear_kernel(LinArgs<T> a)
{
    typedef typename Elem16<T>::vec8 vec8;
    constexpr int kTiles = MT * NT;
    constexpr int kGroup = kTiles < 64 / NWV ? kTiles : 64 / NWV;     // tiles reduced per pass: <= 64 KB of LDS
    static_assert(kTiles % kGroup == 0, "tile groups must divide the tiles");
    __shared__ f32x4 s_part[NWV][kGroup][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int n0 = (int)blockIdx.x * (16 * NT);

    // this wave's share of the k-steps (32 wide); the host guarantees it lies within one product
    const int ks1 = a.K1 >> 5, ks = ks1 + (a.K2 >> 5);
    const int kb = (int)((long long)ks * wave / NWV), ke = (int)((long long)ks * (wave + 1) / NWV);
    const bool second = kb >= ks1;
    const T *wbase = second ? a.w2 : a.w1;
    const int K = second ? a.K2 : a.K1;
    const int k_first = (second ? kb - ks1 : kb) * 32, steps = ke - kb;
    const T *xbase = second ? a.x2 : a.x1;
    const int32_t *map = second ? a.map2 : a.map1;
    const int ldx = second ? a.ldx2 : a.ldx1;

    const T *wp[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (TILED) {                                            // tile (n/16, k/32): 64 lanes x 8 elements, contiguous
            const int ntile = min(n0 / 16 + nt, (a.N + 15) / 16 - 1);
            wp[nt] = wbase + ((size_t)ntile * (K >> 5) + (k_first >> 5)) * 512 + lane * 8;
        } else {
            const int nrow = min(n0 + nt * 16 + r16, a.N - 1);  // rows past N read the last row; never stored
            wp[nt] = wbase + (size_t)nrow * K + k_first + 8 * g;
        }
    }
    const T *xp[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = a.m0 + min(mt * 16 + r16, a.M - 1);
        const size_t row = map ? (size_t)map[m] : (size_t)m * a.mstride;
        xp[mt] = xbase + row * ldx + k_first + 8 * g;
    }
    constexpr int wstep = TILED ? 512 : 32;                     // elements between a lane's vectors of consecutive k-steps
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    constexpr int U = MT + NT <= 3 ? 8 : (MT + NT <= 9 ? 4 : 2);   // k-steps in flight
    int s = 0;
    for (; s + U <= steps; s += U) {
        vec8 wa[U][NT], xb[U][MT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) wa[u][nt] = *reinterpret_cast<const vec8 *>(wp[nt] + (s + u) * wstep);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xb[u][mt] = *reinterpret_cast<const vec8 *>(xp[mt] + (s + u) * 32);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = Elem16<T>::mfma(wa[u][nt], xb[u][mt], acc[mt][nt]);
    }
    for (; s < steps; ++s) {
        vec8 wa[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wa[nt] = *reinterpret_cast<const vec8 *>(wp[nt] + s * wstep);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const vec8 xb = *reinterpret_cast<const vec8 *>(xp[mt] + s * 32);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = Elem16<T>::mfma(wa[nt], xb, acc[mt][nt]);
        }
    }

    // the K shares meet in LDS, a group of tiles at a time; tile j of a group is summed (in wave
    // order, so the result does not depend on timing) and finished by wave j mod NWV
#pragma unroll
    for (int p = 0; p < kTiles / kGroup; ++p) {
        if (p > 0) __syncthreads();
#pragma unroll
        for (int j = 0; j < kGroup; ++j) s_part[wave][j][lane] = acc[(p * kGroup + j) / NT][(p * kGroup + j) % NT];
        __syncthreads();
        for (int j = wave; j < kGroup; j += NWV) {
            f32x4 v = s_part[0][j][lane];
#pragma unroll
            for (int w = 1; w < NWV; ++w) v += s_part[w][j][lane];
            const int id = p * kGroup + j;
            linear_epilogue<T, EPI>(a, v, (id / NT) * 16, n0 + (id % NT) * 16, r16, g);
        }
    }
}

// Layers of up to 8 rows: the stream of the weights and little else.  A workgroup owns 16 columns, its eight waves split K.  A
// unit, two k-steps of 32, is 2 KB of weights and 1 KB of activations, the eight rows of both steps side by side; a wave has three
// units under way, copied from memory straight into its ring in LDS, in operand order, and waits for none but the next.  No
// barrier stands before the waves' sums meet.
//
// What bounds it.  A compute unit has some 64 KB of loads under way, whether they come from HBM or from L2, so activations cost
// what weights do: with a 16-row operand per k-step, as rd_linear_kernel has it, half of all loads are activations, here a third.
// And the memory's channels: where K is a multiple of a power of two, waves that walk their shares in step ask the same few
// channels.  So the workgroups of an XCD start a unit after one another, those of the next XCD two units on, and all of them walk
// around.  us per call (8 x 5 tokens, 32000 tokens, two MLP layers), rd_linear_kernel / this one without the turn / with it:
// hidden size 4096 685 / 669 / 626, 5120 990 / 891 / 895 (another machine: 932), 3072 548 / 488 / 489 (509), 2048 330 / 318 / 316; the output
// layer at 4096 95.8 -> 86.0 us, 6.1 TB/s, an MLP layer 27.0 -> 24.8, 2.5 of it before the first weights arrive.  Turns by the
// plain workgroup number are no substitute (627 to 809 us by the step: workgroups alternate between XCDs).
constexpr int kStreamRows = 8;
constexpr int kStreamWaves = 8, kStreamUnits = 3;      // waves, units a wave has under way: 72 KB of LDS, two workgroups per compute unit
constexpr size_t kStreamLds = (size_t)kStreamWaves * kStreamUnits * 3 * 1024;

template <typename T, int EPI, bool TILED>
__global__ __launch_bounds__(kStreamWaves * 64) void rd_stream_kernel(LinArgs<T> a)
{
    typedef typename Elem16<T>::vec8 vec8;
    constexpr int NWV = kStreamWaves, R = kStreamUnits;
    extern __shared__ __align__(16) unsigned char s_buf[];
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int n0 = (int)blockIdx.x * 16;
    unsigned char *ring = s_buf + wave * (R * 3 * 1024);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)ring;

    // this wave's n units, of one product (where there are two, half of the waves take each); the host guarantees n > 0
    const bool two = a.K2 > 0, second = two && wave >= NWV / 2;
    const int of = two ? NWV / 2 : NWV, at = second ? wave - NWV / 2 : wave;
    const int K = second ? a.K2 : a.K1, units = K >> 6;
    const int ub = units * at / of, n = units * (at + 1) / of - ub;
    const int first = (int)(((blockIdx.x >> 3) + 2 * (blockIdx.x & 7)) % (unsigned)n);      // where it starts
    const T *xbase = second ? a.x2 : a.x1;
    const int32_t *map = second ? a.map2 : a.map1;
    const int m = a.m0 + min(r16 & 7, a.M - 1);         // lanes of r16 < 8 copy the rows' first k-step, the others the second
    const size_t row = map ? (size_t)map[m] : (size_t)m * a.mstride;
    uintptr_t xp = reinterpret_cast<uintptr_t>(xbase + row * (second ? a.ldx2 : a.ldx1) + (size_t)(ub + first) * 64 + (r16 >> 3) * 32 + 8 * g);
    const uintptr_t wbase = reinterpret_cast<uintptr_t>(second ? a.w2 : a.w1);
    uintptr_t wp;
    uint32_t woff;
    constexpr int wstep = TILED ? 1024 : 64;            // bytes between k-steps
    if (TILED) {
        wp = wbase + ((size_t)blockIdx.x * (K >> 5) + (ub + first) * 2) * 1024;
        woff = lane * 16;
    } else {
        wp = wbase + ((size_t)n0 * K + (size_t)(ub + first) * 64) * 2;
        woff = (uint32_t)min(r16, a.N - 1 - n0) * (uint32_t)K * 2 + g * 16;     // rows past N read the last row; never stored
    }
    EpilogueIn in = {};
    if (wave == 0) in = linear_epilogue_in<T, EPI>(a, 0, n0, r16, g);
    int left = n - first;                               // units up to the end of the share
    auto copy = [&](int slot) __attribute__((always_inline)) {
        const uint32_t dst = lds0 + slot * 3072;
        rd::dma16(wp, woff, dst);
        rd::dma16(wp + wstep, woff, dst + 1024);
        rd::dma16(xp, dst + 2048);
        const int next = left == 1 ? 1 - n : 1;
        left = left == 1 ? n : left - 1;
        wp += next * (2 * wstep);
        xp += next * 128;
    };
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u < n) copy(u);
    const int x_rd = (g * 16 + (r16 & 7)) * 16;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int slot = 0;
    for (int u = 0; u < n; ++u) {
        if (u + R <= n) rd::wait_vm<(R - 1) * 3>();
        else rd::wait_vm<0>();
        const unsigned char *p = ring + slot * 3072;
        vec8 w[2], x[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            w[s] = *reinterpret_cast<const vec8 *>(p + s * 1024 + lane * 16);
            x[s] = *reinterpret_cast<const vec8 *>(p + 2048 + x_rd + s * 128);
        }
        rd::wait_lds();
        if (u + R < n) copy(slot);
        slot = slot + 1 == R ? 0 : slot + 1;
        acc = Elem16<T>::mfma(w[0], x[0], acc);
        acc = Elem16<T>::mfma(w[1], x[1], acc);
    }
    // the waves' sums meet in LDS (nothing is under way into it any more) and are added in wave order
    f32x4 *s_part = reinterpret_cast<f32x4 *>(s_buf);
    rd_lds_barrier();
    s_part[wave * 64 + lane] = acc;
    rd_lds_barrier();
    if (wave != 0) return;
    f32x4 v = s_part[lane];
#pragma unroll
    for (int w = 1; w < NWV; ++w) v += s_part[w * 64 + lane];
    linear_epilogue<T, EPI>(a, v, 0, n0, r16, g, in);
}

// Column tiles of weights lie 32 K bytes apart.  Where that is a multiple of 64 KB, workgroups that walk K in step ask the same few
// memory channels, so those of an XCD start one after another and walk around (us per call of 5 positions and two MLP layers
// without / with it, in turn on one machine: 64 rows, hidden size 4096 828 / 781, row-major 900 / 835, 2048 425 / 415, 5120
// 1037 / 1033; 128 rows, 4096 951 / 923; 16 rows, 4096 741 / 719; 80 rows, 1024, 50000 tokens 385 / 362).  Elsewhere the channels
// take turns by themselves, and workgroups that start apart share fewer activations (60 rows, 1536 285 / 294; 32 rows, 6656
// 1346 / 1353), and at 256 rows activations are half of the loads (6656 2060 / 2090).  65 to 128 rows lie between: where K
// is 4096 or less the layers that split K are not turned, the output layer within each XCD only (us per call, no turns / turned as
// fewer rows are / so: 72 rows, 2048 467 / 471 / 461; 1024, 50000 tokens 370 / 342 / 341; larger K as fewer rows: 72 rows, 4096 873 /
// 847, 128 rows, 3072 751 / 742, 5120 1228 / 1212).
__device__ __forceinline__ bool in_phase(int K) { return K % 2048 == 0; }
constexpr int kFarK = 6144;

// The output layer at more than a few rows: with K split over the waves, the accumulators of 128 rows leave
// a workgroup room for only 64 columns, and every workgroup then pulls two activation bytes through the
// caches per weight byte (one per weight byte already at 16 rows, with 16-column workgroups).  Here the waves split the columns instead: a wave owns 32 columns for
// all rows (16 accumulator tiles) and half of every chunk's k-steps, so a workgroup of 8 waves covers 128
// columns with half of the registers (every B operand read from LDS feeds two matrix instructions), all
// waves walk K together in chunks of 256, and the activations of a chunk are staged once per
// workgroup in LDS (row stride 528 bytes: the 16 rows a B-operand read touches fall in distinct banks),
// double-buffered, one barrier per chunk.  Weights still go from memory straight into the A operand, one
// chunk ahead.  An output is the sum of two accumulators, each over its k-steps in the same order for either
// weight layout.
constexpr int kRowsKC = 256;                       // k per chunk
constexpr int kRowsStride = kRowsKC * 2 + 16;      // bytes per staged activation row

template <typename T, int MT, bool TILED>
__global__ __launch_bounds__(512) void rd_head_rows_kernel(LinArgs<T> a)
{
    typedef typename Elem16<T>::vec8 vec8;
    constexpr int kSteps = kRowsKC / 32;                               // k-steps per chunk
    constexpr int kMine = kSteps / 2;                                  // ... of which a wave takes half
    constexpr int kBuf = MT * 16 * kRowsStride;                        // bytes per buffer
    constexpr int kPieces = MT * 16 * (kRowsKC * 2 / 16) / 512;        // 16-byte pieces per thread and chunk
    extern __shared__ __align__(16) unsigned char s_x[];               // two buffers
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cp = wave & 3, kh = wave >> 2;                           // column pair, half of every chunk's k-steps
    const int r16 = lane & 15, g = lane >> 4;
    const int group = (int)blockIdx.x;
    const int n_tile = (group * 8 + cp * 2) * 16;                      // this wave's 32 columns: tiles n_tile, n_tile + 16
    const int nchunks = a.K1 / kRowsKC;
    const unsigned apart = MT > 4 && a.K1 < kFarK ? 0 : 3;          // chunks that an XCD's workgroups start after the last one's
    const int turn = in_phase(a.K1) ? (int)(((blockIdx.x >> 3) + apart * (blockIdx.x & 7)) % (unsigned)nchunks) : 0;      // the chunk it starts with

    const T *wp[2];                                                    // this lane's first weight vector of either tile
    constexpr int wstep = TILED ? 512 : 32;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (TILED) {
            const int ntile = min(n_tile / 16 + t, (a.N + 15) / 16 - 1);   // tiles past N read the last one; never stored
            wp[t] = a.w1 + (size_t)ntile * (a.K1 >> 5) * 512 + lane * 8 + kh * kMine * wstep;
        } else {
            wp[t] = a.w1 + (size_t)min(n_tile + t * 16 + r16, a.N - 1) * a.K1 + 8 * g + kh * kMine * wstep;
        }
    }
    const T *xsrc[kPieces];
    int xdst[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int p = tid + 512 * i, row = p >> 5, ch = p & 31;
        const size_t prow = (size_t)(a.m0 + min(row, a.M - 1)) * a.mstride;
        xsrc[i] = a.x1 + prow * a.ldx1 + ch * 8;
        xdst[i] = row * kRowsStride + ch * 16;
    }
    f32x4 acc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][0] = acc[mt][1] = f32x4{0.f, 0.f, 0.f, 0.f};

    // (staged values are kept as native vectors: arrays of those stay in registers)
    vec8 wa0[2][kMine], wa1[2][kMine];
    {   // the first chunk: activations -> buffer 0, weights -> wa0
        vec8 x0[kPieces];
#pragma unroll
        for (int i = 0; i < kPieces; ++i) x0[i] = *reinterpret_cast<const vec8 *>(xsrc[i] + turn * kRowsKC);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < kMine; ++s) wa0[t][s] = *reinterpret_cast<const vec8 *>(wp[t] + (turn * kSteps + s) * wstep);
#pragma unroll
        for (int i = 0; i < kPieces; ++i) *reinterpret_cast<vec8 *>(s_x + xdst[i]) = x0[i];
    }

    const int b_off = r16 * kRowsStride + g * 16 + kh * kMine * 64;    // B operand: row r16 of a tile, k group g, own k-steps
    auto chunk = [&](int c, vec8 (&cur)[2][kMine], vec8 (&nxt)[2][kMine]) __attribute__((always_inline)) {
        // the next chunk's activations and weights (after the last chunk: the last chunk again, ignored)
        const int next = min(c + 1, nchunks - 1) + turn, cn = next >= nchunks ? next - nchunks : next;
        vec8 xs[kPieces];
#pragma unroll
        for (int i = 0; i < kPieces; ++i) xs[i] = *reinterpret_cast<const vec8 *>(xsrc[i] + cn * kRowsKC);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < kMine; ++s) nxt[t][s] = *reinterpret_cast<const vec8 *>(wp[t] + (cn * kSteps + s) * wstep);
        rd_lds_barrier();                                              // buffer c&1 is complete, buffer (c+1)&1 is free
        const unsigned char *buf = s_x + (c & 1) * kBuf + b_off;
#pragma unroll
        for (int s = 0; s < kMine; ++s) {
            vec8 xb[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xb[mt] = *reinterpret_cast<const vec8 *>(buf + mt * 16 * kRowsStride + s * 64);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[mt][0] = Elem16<T>::mfma(cur[0][s], xb[mt], acc[mt][0]);
                acc[mt][1] = Elem16<T>::mfma(cur[1][s], xb[mt], acc[mt][1]);
            }
        }
        unsigned char *dst = s_x + ((c + 1) & 1) * kBuf;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) *reinterpret_cast<vec8 *>(dst + xdst[i]) = xs[i];
    };
    for (int c = 0; c < nchunks; c += 2) {
        chunk(c, wa0, wa1);
        if (c + 1 < nchunks) chunk(c + 1, wa1, wa0);
    }
    // the two halves of k meet in LDS (the staging buffers are free after one more barrier)
    rd_lds_barrier();
    f32x4 *s_acc = reinterpret_cast<f32x4 *>(s_x) + (size_t)cp * MT * 2 * 64 + lane;
    if (kh == 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            s_acc[(mt * 2 + 0) * 64] = acc[mt][0];
            s_acc[(mt * 2 + 1) * 64] = acc[mt][1];
        }
    }
    rd_lds_barrier();
    if (kh == 1) return;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        linear_epilogue<T, EPI_HEAD>(a, acc[mt][0] + s_acc[(mt * 2 + 0) * 64], mt * 16, n_tile, r16, g);
        linear_epilogue<T, EPI_HEAD>(a, acc[mt][1] + s_acc[(mt * 2 + 1) * 64], mt * 16, n_tile + 16, r16, g);
    }
}

// Layers of many rows.  A workgroup of eight waves owns RT row tiles x CT column tiles of the output and a share of K;
// wave (wr, wc) of WR x WC owns a block of RT/WR x CT/WC tiles.  Per k-step of 32 the operands of all its tiles, (RT + CT) KB,
// are copied from memory straight into buffers in LDS, up to one k-step less ahead than there are buffers, with one LDS-only barrier
// a step or two; operands are read into registers two row tiles
// ahead, across that barrier.  K is split over a.ksplit workgroups; each leaves its tiles in the workspace and
// rd_linear_finish_kernel adds them up in split order.  Workgroups of one split read the same activations: an XCD gets
// consecutive column groups of one split.
//
// What bounds it.  64 and 128 rows: what a compute unit has under way, weights and activations together, 4.7 to 5.2 TB/s of
// weights (the MLP layer at a hidden size of 5120 40 to 45 us by the machine, and 5 of adding up).  256 rows: a k-step takes 1750 to
// 1800 clocks where its matrix instructions take 1024.  The copies take part of the rest (the output layer at a hidden size of
// 6656 217 us, 180 with the activations' alone, 200 with the weights', 145 with none, at a clock that the matrix cores' power
// holds at 1.75 to 1.9 GHz; a library product of 8192^3 reaches 1.22 PFLOP/s), but not by their traffic in LDS: with weights straight
// into registers, half of it, a call is 2 % longer.  Against the kernels it replaced, one that
// staged the activations of 128 rows through registers and one that split K over the waves, us per layer: 256 rows, hidden
// size 6656, RNN 137 -> 52 + 14, MLP 173 -> 107 + 18, output layer 297 -> 208 + 17; 64 rows, 5120, RNN 37 -> 24 + 6, MLP 56 ->
// 43 + 6.  A call: 256 rows 2832 -> 2124 (2072 with the selection below), 64 rows 1085 -> 1056 (1018), 80 rows, hidden size 1024 and 50000 tokens 592 -> 465; shapes that the
// old kernels' rules fitted badly gain most (80 rows, hidden size 4160, 12000 tokens 1377 -> 677).
//
// Buffers and rounds.  At 64 rows and fewer the weights that may be under way are kept to what a compute unit has under way, some
// 64 KB; more only queue.  256 columns: two k-steps between barriers, of which there are else so many that the loop takes half the
// time even without its copies.  128 columns: one, and activations seven steps ahead.  us per call, 64 rows of hidden size 5120 / 4096
// / 6656: four buffers of activations, as many of weights as fit, a barrier per k-step 1003 / 802 / 1444; 5 (256 columns) and 8 (128)
// of weights 994 / 778 / 1434; as here 979 / 772 / 1417; two k-steps a round for both 984 / 784 / 1420, four for 128 columns 1029 / 805
// / 1418.  Their numbers are powers of two: 7, 9, 10 or 12 take 5 to 15 us more at 5120.  More rows: as many as fit (two k-steps a round
// at 128 rows, of 5120 1203 -> 1241, of 4096 924 -> 950).
template <int RT, int CT> constexpr int gemm_round() { return RT == 4 && CT == 16 ? 2 : 1; }       // k-steps between two barriers
template <int RT> constexpr int gemm_x_buffers() { return RT == 4 ? 8 : 4; }       // buffers for the activations' k-steps
template <int RT, int CT> constexpr int gemm_w_buffers()                           // ... and for the weights'
{
    return RT == 4 ? 8 : (160 - gemm_x_buffers<RT>() * RT) / CT < 12 ? (160 - gemm_x_buffers<RT>() * RT) / CT : 12;
}
template <int RT, int CT> constexpr bool gemm_trims() { return CT == 16 && RT < 16; }       // may have 13 to 15 column tiles (TRIM)
template <int RT, int CT> constexpr size_t gemm_lds() { return (size_t)(gemm_x_buffers<RT>() * RT + gemm_w_buffers<RT, CT>() * CT) * 1024; }

template <typename T, int RT, int CT, int WR, int WC, int EPI, bool TILED, bool TRIM>
__global__ __launch_bounds__(WR * WC * 64, 1) void rd_gemm_kernel(LinArgs<T> a)
{
    typedef typename Elem16<T>::vec8 vec8;
    constexpr int KU = gemm_round<RT, CT>(), NX = gemm_x_buffers<RT>(), NW = gemm_w_buffers<RT, CT>(), RX = NX / KU, RW = NW / KU;
    constexpr int PX = (RT + 3) / 4, PW = CT / 4;                       // 1 KB pieces a wave copies per k-step: four waves X, four W
    constexpr int MT = RT / WR, NT = CT / WC;                           // a wave's tiles
    static_assert(WR * WC == 8 && CT % 4 == 0 && MT % 2 == 0 && NT % (MT / 2) == 0, "whole pieces, and halves of a step");
    static_assert(NX % KU == 0 && NW % KU == 0 && RX >= 3 && RW >= 3, "whole rounds, one of them under way");
    extern __shared__ __align__(16) unsigned char s_buf[];
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)s_buf;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int cols = TRIM ? a.cols : CT;                                // column tiles of the CT that are there; the others' products are ignored
    const int groups = (a.N + 16 * cols - 1) / (16 * cols);
    const int unit = (int)(blockIdx.x & 7) * ((int)gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    if (unit >= groups * a.ksplit) return;
    const int split = unit / groups, group = unit - split * groups;
    const int n0 = group * (16 * cols);

    // this workgroup's k-steps: [kb, ke) of those of the first product and, behind them, of the second
    const int ks1 = a.K1 >> 5, ks = ks1 + (a.K2 >> 5);
    const int kb = (int)((long long)ks * split / a.ksplit), steps = (int)((long long)ks * (split + 1) / a.ksplit) - kb;
    const int turn = (RT < 8 || (RT == 8 && a.K1 >= kFarK)) && in_phase(a.K1) && steps > 0 ? (int)((blockIdx.x >> 3) * 3 % (unsigned)steps) : 0;      // where it starts
    auto kstep = [&](int s) __attribute__((always_inline)) {
        const int t = min(s, steps - 1) + turn;
        return kb + (t >= steps ? t - steps : t);
    };

    // A wave's pieces: the first four waves copy row tiles wave, wave + 4, .. of the activations (past the last: that one
    // again, to the same place), the others column tiles of the weights.  (Loads return in order: a wave that copied both would
    // wait for its newest weights whenever it waits for activations.)  Rows are copied four lanes to a row (64 bytes of it);
    // the 16-byte pieces of a row are swizzled so that the 16 rows of an operand read lie in distinct banks.
    const bool is_x = wave < 4;
    const bool whole = !TRIM || (wave & 3) + 4 * (PW - 1) < cols;       // else one piece of the weights fewer
    const int wq = wave & 3, prow = lane >> 2, pch = (lane & 3) ^ (prow >> 2);
    uintptr_t row_at1[PX], row_at2[PX];         // activations: a lane's row in either product
    uint32_t woff[PW];
    int wtile[PW];
    if (is_x) {
        int row1[PX], row2[PX];
#pragma unroll
        for (int i = 0; i < PX; ++i) row1[i] = row2[i] = a.m0 + min(min(wq + 4 * i, RT - 1) * 16 + prow, a.M - 1);
        if (a.map1 != nullptr) {                // (the RNN: both products have one)
            int m1[PX], m2[PX];
#pragma unroll
            for (int i = 0; i < PX; ++i) { m1[i] = a.map1[row1[i]]; m2[i] = a.map2[row2[i]]; }
#pragma unroll
            for (int i = 0; i < PX; ++i) { row1[i] = m1[i]; row2[i] = m2[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < PX; ++i) row1[i] *= a.mstride;
        }
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            row_at1[i] = reinterpret_cast<uintptr_t>(a.x1) + ((size_t)row1[i] * a.ldx1 + pch * 8) * 2;
            row_at2[i] = reinterpret_cast<uintptr_t>(a.x2) + ((size_t)row2[i] * a.ldx2 + pch * 8) * 2;
        }
    } else {
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            wtile[i] = min(n0 / 16 + wq + 4 * i, (a.N + 15) / 16 - 1);  // past N: the last one again; never stored
            woff[i] = TILED ? lane * 16 : (uint32_t)min((wq + 4 * i) * 16 + prow, a.N - 1 - n0);      // row-major: of the row in the group
        }
    }
    const uintptr_t w1 = reinterpret_cast<uintptr_t>(a.w1), w2 = reinterpret_cast<uintptr_t>(a.w2);
    auto copy_x = [&](int s) __attribute__((always_inline)) {
        const int k = kstep(s);
        const bool second = k >= ks1;
        const size_t at = (size_t)(second ? k - ks1 : k) * 64;
#pragma unroll
        for (int i = 0; i < PX; ++i) rd::dma16((second ? row_at2[i] : row_at1[i]) + at, lds0 + ((uint32_t)(s % NX) * RT + min(wq + 4 * i, RT - 1)) * 1024);
    };
    auto copy_w = [&](int s) __attribute__((always_inline)) {
        const int k = kstep(s);
        const bool second = k >= ks1;
        const int k1 = second ? k - ks1 : k, K = second ? a.K2 : a.K1;
        const uintptr_t wb = second ? w2 : w1;
        const uint32_t dst = lds0 + (NX * RT + (uint32_t)(s % NW) * CT + wq) * 1024;
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            if (i == PW - 1 && !whole) break;
            if (TILED) rd::dma16(wb + ((size_t)wtile[i] * (K >> 5) + k1) * 1024, woff[i], dst + 4 * i * 1024);
            else rd::dma16(wb + ((size_t)n0 * K + (size_t)k1 * 32) * 2, woff[i] * (uint32_t)K * 2 + pch * 16, dst + 4 * i * 1024);
        }
    };

    const int wr = wave / WC, wc = wave % WC;
    const int rd_rows = r16 * 64 + (g ^ (r16 >> 2)) * 16;               // operand order from copied rows
    const int rd_w = NX * RT * 1024 + wc * NT * 1024 + (TILED ? lane * 16 : rd_rows), rd_x = wr * MT * 1024 + rd_rows;
    auto read_w = [&](int s, int nt) __attribute__((always_inline)) { return *reinterpret_cast<const vec8 *>(s_buf + (s % NW) * (CT * 1024) + rd_w + nt * 1024); };
    auto read_x = [&](int s, int mt) __attribute__((always_inline)) { return *reinterpret_cast<const vec8 *>(s_buf + (s % NX) * (RT * 1024) + rd_x + mt * 1024); };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Rounds of KU k-steps (where the last one is not whole, its last k-step again).
    const int rounds = (steps + KU - 1) / KU;
    auto copy_round = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            if (is_x) copy_x(r * KU + u);
            else copy_w(r * KU + u);
        }
    };
    for (int r = 0; r < min(rounds, (is_x ? RX : RW) - 1); ++r) copy_round(r);
    // round r, behind which at most RX - 3 (RW - 3) more are asked for, is in LDS when all waves have waited for their pieces of it
    auto arrive = [&](int r) __attribute__((always_inline)) {
        if (is_x) {
            if (r + RX - 3 < rounds) rd::wait_vm<(RX - 3) * KU * PX>();
            else rd::wait_vm<0>();
        } else {
            if (r + RW - 3 >= rounds) rd::wait_vm<0>();
            else if (whole) rd::wait_vm<(RW - 3) * KU * PW>();
            else rd::wait_vm<(RW - 3) * KU * (PW - 1)>();
        }
        rd_lds_barrier();
    };
    // One k-step, a row tile at a time.  A row tile's operand is read two row tiles ahead, the next step's weights in the
    // second half (after the last step: what lies there, ignored).
    vec8 x[MT];
    auto step = [&](int s, const vec8 (&w)[NT], vec8 (&wn)[NT]) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            constexpr int kHalf = MT / 2;
            if (mt == kHalf - 1 && s + 1 < steps && (s + 1) % KU == 0) {
                const int r = (s + 1) / KU, ahead = r + (is_x ? RX : RW) - 2;
                arrive(r);                    // (all waves have read the round before the one that ends here: its buffers are free)
                if (ahead < rounds) copy_round(ahead);
            }
            const vec8 xm = x[mt];
            x[(mt + 2) % MT] = mt + 2 < MT ? read_x(s, mt + 2) : read_x(s + 1, mt + 2 - MT);
            if (mt >= kHalf) {
#pragma unroll
                for (int i = 0; i < NT / kHalf; ++i) wn[(mt - kHalf) * (NT / kHalf) + i] = read_w(s + 1, (mt - kHalf) * (NT / kHalf) + i);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = Elem16<T>::mfma(w[nt], xm, acc[mt][nt]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (steps > 0) {
        vec8 w0[NT], w1r[NT];
        arrive(0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) w0[nt] = read_w(0, nt);
        x[0] = read_x(0, 0);
        x[1] = read_x(0, 1);
        int s = 0;
        for (; s + 2 <= steps; s += 2) {
            step(s, w0, w1r);
            step(s + 1, w1r, w0);
        }
        if (s < steps) step(s, w0, w1r);
    }
    if (a.ksplit == 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (wc * NT + nt < cols) linear_epilogue<T, EPI>(a, acc[mt][nt], (wr * MT + mt) * 16, n0 + (wc * NT + nt) * 16, r16, g);
        return;
    }
    // tiles numbered as an RT x CT grid
    float *out = a.kpart + ((size_t)group * a.ksplit + split) * (RT * CT) * 256 + lane * 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if ((wr * MT + mt) * 16 < a.M && wc * NT + nt < cols) *reinterpret_cast<f32x4 *>(out + ((wr * MT + mt) * CT + wc * NT + nt) * 256) = acc[mt][nt];
}

// Adds the partial tiles of rd_gemm_kernel in split order and finishes the layer, a wave per tile.  Short layers are bound by
// their round trips: the arguments are fetched together, skip input and bias beside the partial sums.
template <typename T, int RT, int CT, int EPI, bool TRIM>
__global__ __launch_bounds__(256) void rd_linear_finish_kernel(LinArgs<T> a)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    asm volatile("" : : "s"(a.kpart), "s"(a.ksplit), "s"(a.cols), "s"(a.M), "s"(a.N), "s"(a.m0), "s"(a.mstride), "s"(a.bias), "s"(a.res), "s"(a.ldy),
                 "s"(a.y_f32), "s"(a.y_bf), "s"(a.s_bf));
    const int nts = (a.N + 15) / 16, id = blockIdx.x * 4 + wave;
    const int mt = id / nts, n_tile = id - mt * nts;
    if (mt * 16 >= a.M) return;
    const EpilogueIn in = linear_epilogue_in<T, EPI>(a, mt * 16, n_tile * 16, lane & 15, lane >> 4);
    const int cols = TRIM ? a.cols : CT, group = n_tile / cols;
    const float *src = a.kpart + (((size_t)group * a.ksplit * RT + mt) * CT + (n_tile - group * cols)) * 256 + lane * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < a.ksplit; s0 += 8) {
        f32x4 p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = *reinterpret_cast<const f32x4 *>(src + (size_t)min(s0 + i, a.ksplit - 1) * (RT * CT) * 256);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (s0 + i < a.ksplit) v += p[i];
    }
    linear_epilogue<T, EPI>(a, v, mt * 16, n_tile * 16, lane & 15, lane >> 4, in);
}

// rows m = b*W + w: X0 = [e(last token), h] (fp32 and bf16), state = e(last token), path = [last token].  The first position
// computes one row per sequence, w = 0, and later ones write their own states: e only goes there.  A workgroup takes 2048
// elements of a row, so that each lane has one load of e and one of h to wait for (256 rows of hidden size 6656: 14.3 -> 7.7 us,
// 64 rows of 5120 8.6 -> 5.1).
template <typename T>
__global__ void rd_draft_init_kernel(const T *__restrict__ emb, const T *__restrict__ h,
                                     const int32_t *__restrict__ last_token, int W, int L, int Dm, int V,
                                     float *__restrict__ x_f32, T *__restrict__ x_bf, T *__restrict__ s_bf,
                                     int32_t *__restrict__ paths, float *__restrict__ cum)
{
    const int m = blockIdx.x, b = m / W;
    int tok = last_token[b];
    tok = tok < 0 ? 0 : (tok > V - 1 ? V - 1 : tok);
    const bool first = m % W == 0;                                        // uniform
    const int i = (blockIdx.y * blockDim.x + threadIdx.x) * 8;
    if (i < Dm) {                                                         // Dm is a multiple of 64
        typedef typename Elem16<T>::vec8 vec8;
        const vec8 hv = *reinterpret_cast<const vec8 *>(h + (size_t)b * Dm + i);
        *reinterpret_cast<vec8 *>(x_bf + (size_t)m * 2 * Dm + Dm + i) = hv;
#pragma unroll
        for (int j = 0; j < 8; ++j) x_f32[(size_t)m * 2 * Dm + Dm + i + j] = (float)hv[j];
        if (first) {
            const vec8 e = *reinterpret_cast<const vec8 *>(emb + (size_t)tok * Dm + i);
            *reinterpret_cast<vec8 *>(x_bf + (size_t)m * 2 * Dm + i) = e;
            *reinterpret_cast<vec8 *>(s_bf + (size_t)m * Dm + i) = e;
#pragma unroll
            for (int j = 0; j < 8; ++j) x_f32[(size_t)m * 2 * Dm + i + j] = (float)e[j];
        }
    }
    if (blockIdx.y == 0) {
        for (int j = threadIdx.x; j < L; j += blockDim.x) paths[(size_t)m * L + j] = tok;
        if (threadIdx.x == 0) cum[m] = 0.f;
    }
}

__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// Selection beyond kFewBeam candidates is a merge of sorted lists, one list per lane: every round the lanes offer
// the heads of their lists, the largest value wins and, among equal values, the lowest lane (lists are
// laid out so that a lower lane means a smaller candidate or smaller tokens, which is the tie rule).
// A round is a maximum over lanes by data-parallel primitives, a ballot and a find-first-set; only the
// winning lane fetches a new head.
template <int kCtrl>
__device__ __forceinline__ float max_step_dpp(float x)
{
    return fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), kCtrl, 0xf, 0xf, false)));
}
// maximum over each group of 8 consecutive lanes
__device__ __forceinline__ float group8_max(float x)
{
    x = max_step_dpp<0xB1>(x);          // quad_perm [1,0,3,2]: partner lane ^ 1
    x = max_step_dpp<0x4E>(x);          // quad_perm [2,3,0,1]: partner lane ^ 2
    return max_step_dpp<0x141>(x);      // row_half_mirror: the other quad of the 8
}
// maximum over the 64 lanes, the same value in every lane
__device__ __forceinline__ float wave_max(float x)
{
    x = max_step_dpp<0x140>(group8_max(x));                 // row_mirror: the other half of the 16
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
// lowest lane of the wave whose `offer` is set, -1 if none (uniform)
__device__ __forceinline__ int first_lane(bool offer)
{
    const unsigned long long m = __ballot(offer);
    return m ? __ffsll((long long)m) - 1 : -1;
}

constexpr int kChunk = 4096;            // logits per workgroup of the first top-W pass
constexpr int kChunkThreads = 256;
constexpr int kChunkPer = kChunk / kChunkThreads;
static_assert(kMaxVocab / kChunk <= 64, "one lane per chunk in the row pass");

// Compare-exchange of a sorting network on (value, position) pairs: the better pair goes to a.
__device__ __forceinline__ void order_pair(float &va, int &ka, float &vb, int &kb)
{
    const bool swap = better(vb, kb, va, ka);
    const float tv = swap ? vb : va, uv = swap ? va : vb;
    const int tk = swap ? kb : ka, uk = swap ? ka : kb;
    va = tv; vb = uv; ka = tk; kb = uk;
}

// First pass for up to 28 candidates, the same results: workgroup (chunk c, row m).  No list is sorted: the W-th best of the
// maxima of 32 groups of logits is a lower bound of the chunk's W-th best logit, few logits but the W best reach it (some 1.2 W
// of them in random rows), and those are ranked by counting how many of them are better.  A group is eight lanes; a lane owns
// four quads of tokens, or, in a chunk of up to 1024, four tokens one by one, so that no group is empty where there are more
// than 256 tokens.  Bound by vector instructions (256 rows of 32000 logits, eight workgroups per compute unit: 12.0 us, with
// every lane's tokens sorted as below 19.1; 8 rows 5.6 and 8.2).  Where more than 512 logits reach the bound, equal ones as a
// rule, those equal to it are numbered in the order of their tokens and only as many taken as are missing (112 rows of 32000 equal
// logits, 28 candidates, 14 us; 48 by the rounds that follow).  Where more than 512 are larger than it, or a row holds NaN or
// +inf, W rounds pick the best one left.
__global__ __launch_bounds__(kChunkThreads) void rd_topw_few_kernel(const float *__restrict__ logits, int V, int W, int chunks, int mstride,
                                                                    float *__restrict__ part_max, float *__restrict__ part_sum,
                                                                    float *__restrict__ part_cv, int32_t *__restrict__ part_ci)
{
    constexpr int kWaves = kChunkThreads / 64, kGroups = 32, kCap = 2 * kChunkThreads;
    static_assert(kGroups * 8 == kChunkThreads && kFewBeam <= kGroups, "a group is eight lanes");
    __shared__ float s_g[kGroups], s_v[kWaves];
    __shared__ __align__(16) uint2 s_c[kCap];               // (logit, token) of those that reach the bound
    __shared__ float s_cv[kWaves][kFewBeam];
    __shared__ int s_ci[kWaves][kFewBeam];
    __shared__ int s_n, s_eq[4][kWaves];
    const int c = blockIdx.x, m = blockIdx.y * mstride, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *z = logits + (size_t)m * V;
    // this lane's token j is t0 + (j / 4) * far + (j % 4) * near, none from V on
    const bool quads = V - c * kChunk > 4 * kChunkThreads;              // uniform
    const int t0 = c * kChunk + tid * (quads ? 4 : 1), far = quads ? 4 * kChunkThreads : kMaxVocab, near = quads ? 1 : kChunkThreads;
    auto token = [&](int j) __attribute__((always_inline)) { return t0 + (j >> 2) * far + (j & 3) * near; };
    float x[kChunkPer];
    if ((c + 1) * kChunk <= V) {
#pragma unroll
        for (int j = 0; j < kChunkPer; j += 4) {
            const rd::f4_any q = *reinterpret_cast<const rd::f4_any *>(z + token(j));
            x[j] = q[0]; x[j + 1] = q[1]; x[j + 2] = q[2]; x[j + 3] = q[3];
        }
    } else {
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) x[j] = z[min(token(j), V - 1)];
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) x[j] = token(j) < V ? x[j] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) mx = fmaxf(mx, x[j]);
    mx = group8_max(mx);
    if ((lane & 7) == 0) s_g[tid >> 3] = mx;
    s_c[tid] = s_c[tid + kChunkThreads] = make_uint2(__float_as_uint(-INFINITY), 0x7fffffffu);     // (past the last: lose every comparison)
    if (tid == 0) s_n = 0;
    __syncthreads();
    const float g = s_g[lane & (kGroups - 1)];
    mx = wave_max(g);
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) sum += token(j) < V ? __expf(x[j] - mx) : 0.f;
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == 0) s_v[wave] = sum;
    // the bound: the group maximum that W - 1 others precede (lanes 32 and up repeat the lower ones)
    int before = 0;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g), i));
        before += (o > g || (o == g && i < (lane & (kGroups - 1)))) ? 1 : 0;
    }
    const int at = first_lane(before == W - 1);             // (none only among NaN)
    const float bound = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g), at < 0 ? 0 : at));
    int mine = 0;
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) mine += (token(j) < V && x[j] >= bound) ? 1 : 0;
    if (mine > 0) {
        int pos = atomicAdd(&s_n, mine);
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) {
            if (token(j) < V && x[j] >= bound) {
                if (pos < kCap) s_c[pos] = make_uint2(__float_as_uint(x[j]), (unsigned)token(j));
                ++pos;
            }
        }
    }
    __syncthreads();
    const size_t slot = (size_t)m * chunks + c;
    const float total = s_v[0] + s_v[1] + s_v[2] + s_v[3];
    int n = s_n;
    if (tid == 0) {
        part_max[slot] = mx;
        part_sum[slot] = total;
    }
    if (__builtin_expect(n > kCap && total == total, 0)) { // uniform (out of the way of the rest)
        unsigned equal = 0, larger = 0;                     // this lane's tokens that are
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) {
            equal |= (token(j) < V && x[j] == bound ? 1u : 0u) << j;
            larger |= (token(j) < V && x[j] > bound ? 1u : 0u) << j;
        }
        // Tokens in their order: by quad, then lane, then place in the quad; of a short chunk by j, then lane.
        auto is_equal = [&](int q, int u) __attribute__((always_inline)) { return (quads ? equal >> (4 * q + u) : u == 0 ? equal >> q : 0u) & 1u; };
        int lower[4];                                       // equal ones of the lanes before this one in the wave, by quad
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int all = 0;
            lower[q] = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long b = __ballot(is_equal(q, u));
                all += __popcll(b);
                lower[q] += __popcll(b & ((1ull << lane) - 1));
            }
            if (lane == 0) s_eq[q][wave] = all;
        }
        __syncthreads();                                    // (all have read s_n)
        s_c[tid] = s_c[tid + kChunkThreads] = make_uint2(__float_as_uint(-INFINITY), 0x7fffffffu);
        if (tid == 0) s_n = 0;
        __syncthreads();
        int pos = larger ? atomicAdd(&s_n, __popc(larger)) : 0;
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) {
            if (larger >> j & 1u) {
                if (pos < kCap) s_c[pos] = make_uint2(__float_as_uint(x[j]), (unsigned)token(j));
                ++pos;
            }
        }
        __syncthreads();
        const int n_larger = s_n, missing = max(W - n_larger, 0);
        int first = 0;                                      // equal ones before this wave's in the quad
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int at = first + lower[q];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                at += w < wave ? s_eq[q][w] : 0;
                first += s_eq[q][w];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (is_equal(q, u)) {
                    if (at < missing) s_c[n_larger + at] = make_uint2(__float_as_uint(bound), (unsigned)(quads ? token(4 * q + u) : token(q)));
                    ++at;
                }
            }
        }
        __syncthreads();
        n = n_larger + missing;
    }
    if (n <= kCap && total == total) {                      // uniform
        for (int i = tid; i < n; i += kChunkThreads) {
            const uint2 e = s_c[i];
            const float ev = __uint_as_float(e.x);
            int rank = 0;
            for (int k = 0; k < n; k += 8) {
#pragma unroll
                for (int u = 0; u < 8; u += 2) {
                    const uint4 o = *reinterpret_cast<const uint4 *>(&s_c[k + u]);
                    rank += better(__uint_as_float(o.x), (int)o.y, ev, (int)e.y) ? 1 : 0;
                    rank += better(__uint_as_float(o.z), (int)o.w, ev, (int)e.y) ? 1 : 0;
                }
            }
            if (rank < W) {
                part_cv[slot * W + rank] = ev;
                part_ci[slot * W + rank] = (int)e.y;
            }
        }
        if (tid >= n && tid < W) {                          // fewer than W tokens in the chunk
            part_cv[slot * W + tid] = -INFINITY;
            part_ci[slot * W + tid] = 0x7fffffff;
        }
        return;
    }
    unsigned left = 0;                                      // this lane's tokens not yet picked
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) left |= (token(j) < V ? 1u : 0u) << j;
    for (int r = 0; r < W; ++r) {
        float hv = -INFINITY;
        int hj = kChunkPer, ht = 0x7fffffff;
#pragma unroll
        for (int j = kChunkPer - 1; j >= 0; --j)
            if ((left >> j & 1u) && x[j] >= hv) { hv = x[j]; hj = j; ht = token(j); }
        const float best = wave_max(hv);
        const int tok = (int)rd::wave_reduce_min_u(hv == best ? (unsigned)ht : 0x7fffffffu);
        if (lane == 0) { s_cv[wave][r] = best; s_ci[wave][r] = tok; }
        if (hj < kChunkPer && ht == tok) left &= ~(1u << hj);
    }
    __syncthreads();
    // the four waves' lists: an entry's place is the number of better ones; all entries differ in their token but the
    // fillers, which come last
    for (int i = tid; i < kWaves * W; i += kChunkThreads) {
        const int w = i / W, r = i - w * W, tok = s_ci[w][r];
        const float v = s_cv[w][r];
        int place = 0;
#pragma unroll
        for (int kw = 0; kw < kWaves; ++kw) {
            for (int kr = 0; kr < W; ++kr) {
                const int ot = s_ci[kw][kr];
                place += better(s_cv[kw][kr], ot, v, tok) || (ot == tok && kw * W + kr < i) ? 1 : 0;
            }
        }
        if (place < W) {
            part_cv[slot * W + place] = v;
            part_ci[slot * W + place] = tok;
        }
    }
}

// First pass for more candidates: workgroup (chunk c, row m) reduces 4096 logits to their maximum, the
// sum of exp(x - maximum) and their W best (value, then smaller token).  A lane owns 16 consecutive
// tokens and sorts them in registers (odd-even merge sort network); the sorted lists go to LDS.  Each
// wave merges its 64 lists into its W best, wave 0 then merges the four waves' lists.
__global__ __launch_bounds__(kChunkThreads) void rd_topw_chunk_kernel(const float *__restrict__ logits, int V, int W, int chunks, int mstride, int lpc,
                                                                      float *__restrict__ part_max, float *__restrict__ part_sum,
                                                                      float *__restrict__ part_cv, int32_t *__restrict__ part_ci)
{
    constexpr int kWaves = kChunkThreads / 64;
    __shared__ float s_v[kWaves];
    __shared__ float s_mx;
    __shared__ float s_lv[kChunkPer][kChunkThreads];        // sorted lists, position-major (a lane's column)
    __shared__ unsigned char s_lk[kChunkPer][kChunkThreads];
    __shared__ float s_cv[kWaves][kMaxBeam];
    __shared__ int s_ci[kWaves][kMaxBeam];
    const int c = blockIdx.x, m = blockIdx.y * mstride, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *z = logits + (size_t)m * V;
    const int t0 = c * kChunk + tid * kChunkPer;            // this lane's first token
    float x[kChunkPer];
    int k[kChunkPer];
    if (t0 + kChunkPer <= V) {
#pragma unroll
        for (int j = 0; j < kChunkPer; j += 4) {
            const rd::f4_any q = *reinterpret_cast<const rd::f4_any *>(z + t0 + j);
            x[j] = q[0]; x[j + 1] = q[1]; x[j + 2] = q[2]; x[j + 3] = q[3];
        }
    } else {
#pragma unroll
        for (int j = 0; j < kChunkPer; ++j) x[j] = t0 + j < V ? z[t0 + j] : -INFINITY;
    }
    int n_valid = V - t0;
    n_valid = n_valid < 0 ? 0 : (n_valid > kChunkPer ? kChunkPer : n_valid);
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) { k[j] = j; mx = fmaxf(mx, x[j]); }
    mx = wave_max(mx);
    if (lane == 0) s_v[wave] = mx;
    __syncthreads();
    if (tid == 0) s_mx = fmaxf(fmaxf(s_v[0], s_v[1]), fmaxf(s_v[2], s_v[3]));
    __syncthreads();
    mx = s_mx;
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) sum += j < n_valid ? __expf(x[j] - mx) : 0.f;
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    __syncthreads();
    if (lane == 0) s_v[wave] = sum;

    // sort the lane's 16 (value, position) pairs, best first (Batcher's odd-even merge sort);
    // positions past the end of the vocabulary hold -inf and, being later positions, sort behind
    // real tokens of the same value
#pragma unroll
    for (int pp = 1; pp < kChunkPer; pp <<= 1)
#pragma unroll
        for (int kk = pp; kk >= 1; kk >>= 1)
#pragma unroll
            for (int jj = kk % pp; jj + kk < kChunkPer; jj += 2 * kk)
#pragma unroll
                for (int ii = 0; ii < kk; ++ii)
                    if (ii + jj + kk < kChunkPer && (ii + jj) / (2 * pp) == (ii + jj + kk) / (2 * pp))
                        order_pair(x[ii + jj], k[ii + jj], x[ii + jj + kk], k[ii + jj + kk]);
#pragma unroll
    for (int j = 0; j < kChunkPer; ++j) {
        s_lv[j][tid] = x[j];
        s_lk[j][tid] = (unsigned char)k[j];
    }
    // (a lane reads back only its own column: no barrier needed before the merge)

    // merge of the wave's 64 lists.  Every lane keeps its head and the entry behind it in registers, so
    // a winner moves on without waiting for LDS; the read that refills the second register is only
    // waited for when the same lane wins again.
    float hv = n_valid > 0 ? x[0] : -INFINITY, nv = x[1];
    int hk = k[0], nk = k[1], ptr = 0;
    bool live = n_valid > 0;
    for (int r = 0; r < W; ++r) {
        const float best = wave_max(live ? hv : -INFINITY);
        const int win = first_lane(live && hv == best);
        if (win < 0) {                                      // fewer than W tokens in this wave's range
            if (lane == 0) { s_cv[wave][r] = -INFINITY; s_ci[wave][r] = 0x7fffffff; }
            continue;
        }
        const int wk = __builtin_amdgcn_readlane(hk, win);
        if (lane == 0) {
            s_cv[wave][r] = best;
            s_ci[wave][r] = c * kChunk + (wave * 64 + win) * kChunkPer + wk;
        }
        if (lane == win) {
            ++ptr;
            live = ptr < n_valid;
            hv = nv; hk = nk;
            const int nx = ptr + 1 < kChunkPer ? ptr + 1 : kChunkPer - 1;
            nv = s_lv[nx][tid]; nk = s_lk[nx][tid];
        }
    }
    __syncthreads();
    const size_t slot = (size_t)m * chunks + c;
    if (lpc == kChunkThreads / 64) {
        // wide beams: the four waves' lists leave as they are (the row pass merges four times as many
        // lists in the same number of rounds, and the W rounds of the merge below are saved)
        if (tid == 0) {
            part_max[slot] = mx;
            part_sum[slot] = s_v[0] + s_v[1] + s_v[2] + s_v[3];
        }
        for (int r = lane; r < W; r += 64) {
            part_cv[(slot * lpc + wave) * W + r] = s_cv[wave][r];
            part_ci[(slot * lpc + wave) * W + r] = s_ci[wave][r];
        }
        return;
    }
    if (wave != 0) return;
    if (lane == 0) {
        part_max[slot] = mx;
        part_sum[slot] = s_v[0] + s_v[1] + s_v[2] + s_v[3];
    }
    // merge of the four waves' lists (a lower wave holds smaller tokens): lanes 0..3
    int p4 = 0;
    const int l4 = lane & (kWaves - 1);
    float h4 = s_cv[l4][0], n4 = s_cv[l4][W > 1 ? 1 : 0];
    int i4 = s_ci[l4][0], j4 = s_ci[l4][W > 1 ? 1 : 0];
    bool live4 = lane < kWaves && i4 != 0x7fffffff;
    for (int r = 0; r < W; ++r) {
        const float best = wave_max(live4 ? h4 : -INFINITY);
        const int win = first_lane(live4 && h4 == best);
        if (win < 0) {
            if (lane == 0) { part_cv[slot * W + r] = -INFINITY; part_ci[slot * W + r] = 0x7fffffff; }
            continue;
        }
        if (lane == win) {
            part_cv[slot * W + r] = best;
            part_ci[slot * W + r] = i4;
            ++p4;
            h4 = n4; i4 = j4;
            live4 = p4 < W && i4 != 0x7fffffff;
            const int nx = p4 + 1 < W ? p4 + 1 : W - 1;
            n4 = s_cv[l4][nx]; j4 = s_ci[l4][nx];
        }
    }
}

// Second pass, one lane per (row, chunk): the row's log-sum-exp from the chunk partials and its W best
// tokens as a merge of the chunks' sorted lists (a lower chunk holds smaller tokens), written as
// cumulative scores row_score[row][r] = cum[row] + log p(token r), best first, with the tokens beside
// them.  LPR lanes serve a row: 8 (eight rows per wave) while the vocabulary has at most eight chunks,
// else 64 (one row per wave).
template <int LPR, int WMAX>
__global__ __launch_bounds__(kSelThreads) void rd_topw_row_kernel(
    const float *__restrict__ part_max, const float *__restrict__ part_sum, const float *__restrict__ part_cv,
    const int32_t *__restrict__ part_ci, int chunks, int lpc, const float *__restrict__ cum_cur, int W, int n_rows, int mstride,
    float *__restrict__ row_score, int32_t *__restrict__ row_tok)
{
    constexpr int kRows = 64 / LPR;                                   // rows per wave
    __shared__ float s_cv[64 * WMAX];                                 // [row in wave][chunk][W], LPR * WMAX per row
    __shared__ int s_ci[64 * WMAX];
    const int tid = threadIdx.x, lane = tid & 63, g = lane / LPR, c = lane % LPR;
    const int row_l = blockIdx.x * kRows + g;                         // logical row of this lane's group
    const bool row_ok = row_l < n_rows;
    const size_t row = (size_t)(row_ok ? row_l : n_rows - 1) * mstride;
    const int n_lists = chunks * lpc;                                 // sorted lists per row (lpc per chunk), lane c holds list c
    const int n_surv = n_lists * W;
    auto group_max = [](float x) { return LPR == 8 ? group8_max(x) : wave_max(x); };
    // log-sum-exp of the row: sum_c part_sum[c] * exp(part_max[c] - max) (loads issued before the staging below)
    const bool lane_ok = row_ok && c < chunks;
    const float pm = lane_ok ? part_max[row * chunks + c] : -INFINITY;
    const float gm = group_max(pm);
    float ps = lane_ok ? part_sum[row * chunks + c] * __expf(pm - gm) : 0.f;
#pragma unroll
    for (int off = 1; off < LPR; off <<= 1) ps += __shfl_xor(ps, off, 64);
    const float lse = gm + __logf(ps);
    const float base = row_ok ? cum_cur[row] : 0.f;
    // the survivors of the workgroup's rows -> LDS, by all four waves (one wave alone would spend most of
    // the kernel here at wide beams); eight loads per lane in flight together, addresses past the end
    // pulled back (no load sits behind a branch)
    {
        const int rows_here = min(kRows, n_rows - blockIdx.x * kRows);
        const int total = rows_here * n_surv;
        for (int i0 = 0; i0 < total; i0 += kSelThreads * 8) {
            float v[8];
            int ti[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int idx = min(i0 + u * kSelThreads + tid, total - 1);
                const int gg = idx / n_surv, q = idx - gg * n_surv;
                const size_t src = (size_t)(blockIdx.x * kRows + gg) * mstride * n_surv + q;
                v[u] = part_cv[src];
                ti[u] = part_ci[src];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int idx = i0 + u * kSelThreads + tid;
                if (idx < total) {
                    const int gg = idx / n_surv, q = idx - gg * n_surv;
                    s_cv[gg * LPR * WMAX + q] = v[u];
                    s_ci[gg * LPR * WMAX + q] = ti[u];
                }
            }
        }
    }
    __syncthreads();
    if (tid >= 64) return;                                            // the merge is one wave's work

    const float *lv = s_cv + g * LPR * WMAX + c * W;                  // this lane's list: chunk c of its row
    const int *li = s_ci + g * LPR * WMAX + c * W;
    int ptr = 0;
    int ht = li[0], nt = li[W > 1 ? 1 : 0];                           // head and the entry behind it, in registers
    float hv = lv[0], nv = lv[W > 1 ? 1 : 0];
    bool live = row_ok && c < n_lists && ht != 0x7fffffff;
    for (int r = 0; r < W; ++r) {
        const float best = group_max(live ? hv : -INFINITY);
        const unsigned long long offers = __ballot(live && hv == best);
        int win;                                                      // chunk that wins in this lane's group
        if (LPR == 8) {
            const unsigned mine = (unsigned)(offers >> (g * 8)) & 0xffu;
            win = mine ? __ffs((int)mine) - 1 : -1;
        } else {
            win = offers ? __ffsll((long long)offers) - 1 : -1;
        }
        if (c == 0 && row_ok) {
            row_score[row * W + r] = win >= 0 ? base + (best - lse) : -INFINITY;
        }
        if (c == win) {
            row_tok[row * W + r] = ht;
            ++ptr;
            hv = nv; ht = nt;
            live = ptr < W && ht != 0x7fffffff;
            const int nx = ptr + 1 < W ? ptr + 1 : W - 1;
            nv = lv[nx]; nt = li[nx];
        } else if (c == 0 && win < 0 && row_ok) {
            row_tok[row * W + r] = 0;
        }
    }
}

// Beam step, one wave per sequence: the best W of the live*W (candidate, token) pairs by cumulative
// score.  Every live row's list is sorted (best first; equal scores by smaller token), so this is a
// merge with lane w holding row w's list: ties go to the smaller candidate, and within a row to the
// list order, i.e. the smaller token.  Then the paths, the scores and the row maps of the next RNN
// update are written.  WIDE (more than 64 candidates): lane w also holds row 64 + w's list, which
// loses ties against every first list, and the lists live in dynamic LDS (2 * live * W words).
template <bool WIDE>
__global__ __launch_bounds__(kSelThreads) void rd_beam_step_kernel(
    const float *__restrict__ row_score, const int32_t *__restrict__ row_tok, int V,
    int W, int L, int t, int live,
    const int32_t *__restrict__ paths_cur, int32_t *__restrict__ paths_next, float *__restrict__ cum_next,
    int32_t *__restrict__ parent_row, int32_t *__restrict__ tok_row,
    int32_t *__restrict__ beams_out, float *__restrict__ logp_out /* both NULL except at the last position */)
{
    constexpr int kCap = WIDE ? kMaxBeam : kNarrowBeam;
    __shared__ float s_score_static[WIDE ? 1 : kNarrowBeam * kNarrowBeam];
    __shared__ int s_ctok_static[WIDE ? 1 : kNarrowBeam * kNarrowBeam];
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ int s_win[kCap], s_tok[kCap], s_ptr[kCap];
    __shared__ float s_winv[kCap];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int n_cand = live * W;
    float *s_score = WIDE ? reinterpret_cast<float *>(s_dyn) : s_score_static;
    int *s_ctok = WIDE ? reinterpret_cast<int *>(s_dyn) + n_cand : s_ctok_static;
    for (int i0 = 0; i0 < n_cand; i0 += kSelThreads * 8) {        // rows b*W .. b*W+live-1 are contiguous
        float v[8];                                               // eight loads per lane in flight together
        int ti[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = min(i0 + u * kSelThreads + tid, n_cand - 1);
            v[u] = row_score[(size_t)b * W * W + idx];
            ti[u] = row_tok[(size_t)b * W * W + idx];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = i0 + u * kSelThreads + tid;
            if (idx < n_cand) { s_score[idx] = v[u]; s_ctok[idx] = ti[u]; }
        }
    }
    __syncthreads();
    if (tid < 64) {                                               // the merge is one wave's work
    // Every lane keeps the head of its list and the entry behind it in registers, so the winner moves
    // on without waiting for LDS; the rounds only record (candidate, position in its list) and the
    // tokens are looked up afterwards, W at a time.
    int ptr = 0, ptr2 = 0;
    bool on = lane < live, on2 = WIDE && lane + 64 < live;
    const int la = (on ? lane : 0) * W, lb = (on2 ? lane + 64 : 0) * W;
    float hv = s_score[la], nv = s_score[la + (W > 1 ? 1 : 0)];
    float hv2 = s_score[lb], nv2 = s_score[lb + (W > 1 ? 1 : 0)];
    for (int r = 0; r < W; ++r) {
        float offer = on ? hv : -INFINITY;
        if (WIDE) offer = fmaxf(offer, on2 ? hv2 : -INFINITY);
        const float best = wave_max(offer);
        int win = first_lane(on && hv == best);
        bool second = false;                                      // the winner is a second list (candidate 64 + lane)
        if (WIDE && win < 0) {
            win = first_lane(on2 && hv2 == best);
            second = win >= 0;
        }
        if (win < 0) win = first_lane(on);                        // NaN scores: keep indices in range
        if (WIDE && win < 0) {
            win = first_lane(on2);
            second = win >= 0;
        }
        if (win < 0) win = 0;
        if (lane == win) {
            s_win[r] = second ? lane + 64 : lane;
            s_winv[r] = best;
            if (WIDE && second) {
                s_ptr[r] = ptr2 < W ? ptr2 : W - 1;
                if (on2) {
                    ++ptr2;
                    on2 = ptr2 < W;
                    hv2 = nv2;
                    nv2 = s_score[lb + (ptr2 + 1 < W ? ptr2 + 1 : W - 1)];
                }
            } else {
                s_ptr[r] = ptr < W ? ptr : W - 1;
                if (on) {                                         // (not so only when no list had anything left to offer)
                    ++ptr;
                    on = ptr < W;
                    hv = nv;
                    nv = s_score[la + (ptr + 1 < W ? ptr + 1 : W - 1)];
                }
            }
        }
    }
    }
    __syncthreads();
    for (int r = tid; r < W; r += kSelThreads) {
        const int tk = s_ctok[s_win[r] * W + s_ptr[r]];
        s_tok[r] = tk < 0 ? 0 : (tk > V - 1 ? V - 1 : tk);
    }
    __syncthreads();
    // candidate r: parent pw = s_win[r], new token s_tok[r]
    for (int i = tid; i < W * L; i += kSelThreads) {
        const int r = i / L, j = i - r * L;
        const int pw = s_win[r];
        const size_t src = ((size_t)b * W + pw) * L;
        const int v = j < t ? paths_cur[src + j] : (j == t ? s_tok[r] : paths_cur[src]);
        paths_next[((size_t)b * W + r) * L + j] = v;
        if (beams_out) beams_out[((size_t)b * W + r) * L + j] = v;
    }
    for (int w = tid; w < W; w += kSelThreads) {
        cum_next[(size_t)b * W + w] = s_winv[w];
        parent_row[(size_t)b * W + w] = b * W + s_win[w];
        tok_row[(size_t)b * W + w] = s_tok[w];
        if (logp_out) logp_out[(size_t)b * W + w] = s_winv[w];
    }
}

// Row pass and beam step in one launch, one workgroup per sequence, for up to 28 candidates whose chunks' lists have a thread
// each (few_lists).  Nothing is merged entry by entry: a thread takes one of the first entries of a list (G lanes to a row), of
// each list as many as make 4 W entries together, and counts how many of these heads score more.  The W first heads are a lower
// bound of the W best entries, a list whose first entry `before` heads precede holds at most W - before of them, and what
// reaches the bound, little more than W entries, is ranked by counting in the whole order: score, then smaller candidate, then
// logit, then smaller token.  Bound by the latency of its chain: loads, the rows' log-sum-exps, five barriers, the stores.
// 64 rows of 16 sequences over 32000 tokens: 9.3 us, as two launches of merges 7.8 + 6.5.
constexpr int kFewLists = 256;
__host__ __device__ inline int few_group(int chunks)                  // lanes of a row: a power of two
{
    int G = 1;
    while (G < chunks) G <<= 1;
    return G;
}
bool few_lists(int W, int chunks) { return W <= kFewBeam && W * few_group(chunks) <= kFewLists; }

__global__ __launch_bounds__(kSelThreads) void rd_row_beam_kernel(
    const float *__restrict__ part_max, const float *__restrict__ part_sum, const float *__restrict__ part_cv,
    const int32_t *__restrict__ part_ci, int chunks, const float *__restrict__ cum_cur, int V, int W, int L, int t, int live,
    const int32_t *__restrict__ paths_cur, int32_t *__restrict__ paths_next, float *__restrict__ cum_next,
    int32_t *__restrict__ parent_row, int32_t *__restrict__ tok_row,
    int32_t *__restrict__ beams_out, float *__restrict__ logp_out /* both NULL except at the last position */)
{
    static_assert(kFewLists == kSelThreads, "a list per thread");
    constexpr int kEntries = kFewBeam * kFewBeam;                     // at most W lists with W entries each
    constexpr int kPaths = 2 * kSelThreads;
    struct Entry { float score, logit; int row, tok; };
    __shared__ __align__(16) float s_head[kFewLists];
    __shared__ __align__(16) Entry s_full[kFewLists], s_e[kEntries];
    __shared__ int s_path[kPaths];
    struct List { int slot, take, row; float base, lse; };
    __shared__ List s_list[kFewBeam];
    __shared__ int s_heads, s_lists, s_n;
    __shared__ unsigned s_bound;
    __shared__ int s_win[kFewBeam], s_tok[kFewBeam];
    __shared__ float s_winv[kFewBeam];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int G = few_group(chunks), per = live * G, depth = tid / per, g = (tid - depth * per) / G, c = tid & (G - 1);
    // as many heads of each list as make kHeads times W of them all, where there are threads for them (W always)
    constexpr int kHeads = 4;
    const int n_lists = live * chunks, n_depth = min(min((kHeads * W + n_lists - 1) / n_lists, W), kFewLists / per);
    const bool mine = c < chunks && depth < n_depth;
    const size_t row0 = (size_t)b * W;                                // rows row0 .. row0+live-1 (at the first position: row0)
    const size_t slot = (row0 + g) * chunks + min(c, chunks - 1);
    float pm[1] = {part_max[slot]}, ps[1] = {part_sum[slot]};
    const float logit = part_cv[slot * W + min(depth, W - 1)];
    const int tok = part_ci[slot * W + min(depth, W - 1)];
    const float base = cum_cur[row0 + g];
    const bool paths_in_lds = W * L <= kPaths;                        // uniform
    int path[2];
    for (int u = 0; u < 2; ++u) path[u] = paths_cur[row0 * L + min(tid + u * kSelThreads, W * L - 1)];
    if (paths_in_lds) { s_path[tid] = path[0]; s_path[tid + kSelThreads] = path[1]; }
    // log-sum-exp of the row: sum_c part_sum[c] * exp(part_max[c] - max)
    auto larger = [](float x, float y) __attribute__((always_inline)) { return fmaxf(x, y); };
    auto plus = [](float x, float y) __attribute__((always_inline)) { return x + y; };
    const float own = c < chunks ? pm[0] : -INFINITY;
    pm[0] = own;
    rd::group_reduce(pm, G, larger);
    ps[0] = c < chunks ? ps[0] * __expf(own - pm[0]) : 0.f;
    rd::group_reduce(ps, G, plus);
    const float lse = pm[0] + __logf(ps[0]);
    if (tid == 0) { s_heads = 0; s_lists = 0; s_n = 0; s_bound = 0xffffffffu; }
    Entry head = {-INFINITY, -INFINITY, 0x7fffffff, 0x7fffffff};      // none: after all others
    const float score = base + (logit - lse);
    const bool on = mine && tok != 0x7fffffff && score == score;      // a row of NaN offers nothing
    if (on) head = {score, logit, g, tok};
    s_head[tid] = head.score;
    s_full[tid] = head;
    __syncthreads();
    const int n_heads = per * n_depth;                                // <= 256
    int before = 0;                                                   // heads of larger score
#pragma unroll 4
    for (int k = 0; k < n_heads; k += 4) {                            // (heads past the last are -inf)
        const float4 h = *reinterpret_cast<const float4 *>(&s_head[k]);
        before += (h.x > head.score ? 1 : 0) + (h.y > head.score ? 1 : 0) + (h.z > head.score ? 1 : 0) + (h.w > head.score ? 1 : 0);
    }
    // scores as unsigned integers in the same order
    auto ordered = [](float x) __attribute__((always_inline)) {
        const unsigned u = __float_as_uint(x + 0.f);                  // (-0 as 0)
        return u & 0x80000000u ? ~u : u | 0x80000000u;
    };
    if (on && before < W) {
        atomicAdd(&s_heads, 1);
        atomicMin(&s_bound, ordered(head.score));
    }
    __syncthreads();
    auto precedes = [](const Entry &x, const Entry &y) __attribute__((always_inline)) {
        const bool same = x.score == y.score, same_row = x.row == y.row;      // (no branches)
        return (x.score > y.score) | (same & ((x.row < y.row) | (same_row & better(x.logit, x.tok, y.logit, y.tok))));
    };
    const unsigned bound = s_heads < W ? 0u : s_bound;                // fewer entries than candidates: every one counts
    if (on && s_heads > W) {                                          // equal scores about the W-th head: by the whole order
        before = 0;
        for (int k = 0; k < n_heads; ++k) before += precedes(s_full[k], head) ? 1 : 0;
    }
    const bool whole = n_depth == W;                                  // uniform: every entry is a head (one candidate as a rule)
    if (on && before < W) {
        if (whole) s_e[atomicAdd(&s_n, 1)] = head;
        else if (depth == 0) s_list[atomicAdd(&s_lists, 1)] = {(int)slot, W - before, g, base, lse};
    }
    __syncthreads();
    const int entries = whole ? 0 : s_lists * W;
    for (int i0 = 0; i0 < entries; i0 += 4 * kSelThreads) {           // (four entries' loads in flight together)
        List list[4];
        float v[4];
        int tk[4];
        bool take[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kSelThreads + tid, l = min(i, entries - 1) / W, r = min(i, entries - 1) - l * W;
            list[u] = s_list[l];
            take[u] = i < entries && r < list[u].take;
            const size_t src = (size_t)list[u].slot * W + r;
            v[u] = part_cv[src];
            tk[u] = part_ci[src];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const Entry e = {list[u].base + (v[u] - list[u].lse), v[u], list[u].row, tk[u]};
            if (take[u] && e.tok != 0x7fffffff && ordered(e.score) >= bound) s_e[atomicAdd(&s_n, 1)] = e;
        }
    }
    if (!whole) __syncthreads();
    const int n = s_n;
    for (int i = tid; i < n; i += kSelThreads) {
        const Entry e = s_e[i];
        int rank = 0;
        for (int k = 0; k < n; k += 4) {                              // (reads in flight; past the last, what lies there, not counted)
            Entry o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = s_e[k + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) rank += ((k + u < n) & precedes(o[u], e)) ? 1 : 0;
        }
        if (rank < W) {
            s_win[rank] = e.row;
            s_winv[rank] = e.score;
            s_tok[rank] = min(max(e.tok, 0), V - 1);
        }
    }
    for (int r = n + tid; r < W; r += kSelThreads) {                  // (keep indices in range)
        s_win[r] = 0;
        s_winv[r] = -INFINITY;
        s_tok[r] = 0;
    }
    if (n == 0) {
        // No row has a score (a logit of +inf, or a whole chunk of -inf, makes its log-sum-exp NaN): the best logits of the
        // first one, as the two kernels above have it.
        __syncthreads();
        const size_t first = row0 * chunks * W;
        for (int i = tid; i < chunks * W; i += kSelThreads) {
            const float v1 = part_cv[first + i];
            const int t1 = part_ci[first + i];
            int rank = 0;
            for (int k = 0; k < chunks * W; ++k) {
                const int t2 = part_ci[first + k];
                rank += better(part_cv[first + k], t2, v1, t1) || (t2 == t1 && k < i) ? 1 : 0;
            }
            if (rank < W && t1 != 0x7fffffff) s_tok[rank] = min(max(t1, 0), V - 1);
        }
    }
    __syncthreads();
    for (int i = tid; i < W * L; i += kSelThreads) {
        const int r = i / L, j = i - r * L;
        const int src = s_win[r] * L + (j < t ? j : 0);
        const int v = j == t ? s_tok[r] : paths_in_lds ? s_path[src] : paths_cur[row0 * L + src];
        paths_next[(row0 + r) * L + j] = v;
        if (beams_out) beams_out[(row0 + r) * L + j] = v;
    }
    for (int w = tid; w < W; w += kSelThreads) {
        cum_next[row0 + w] = s_winv[w];
        parent_row[row0 + w] = (int)row0 + s_win[w];
        tok_row[row0 + w] = s_tok[w];
        if (logp_out) logp_out[row0 + w] = s_winv[w];
    }
}

// For every final candidate, the row of each position's logit matrix that produced its token there:
// follow the parent rows back from the last position.  One thread per candidate.
__global__ void rd_draft_rows_kernel(const int32_t *__restrict__ parents /*[T][M]*/, int M, int W, int T,
                                     int32_t *__restrict__ step_row /*[B][W][T]*/)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    int r = m;
    for (int t = T; t >= 1; --t) {
        r = parents[(size_t)(t - 1) * M + r];
        r = r < 0 ? 0 : (r > M - 1 ? M - 1 : r);
        step_row[(size_t)m * T + t - 1] = r;
    }
}

// Operand-tiled weight layout: the matrix [N][K] (row-major, 16-bit elements) cut into tiles of 16
// rows x 32 columns, tile (n/16, k/32) stored as the 1 KB a wave loads for one MFMA A operand -- lane
// (row n%16, column group g = (k%32)/8) holds its eight consecutive elements at offset lane*8 with
// lane = g*16 + n%16 -- tiles of one row band consecutive in k.  Rows past N are zero.  A wave
// instruction of the linear kernel then reads 1 KB of consecutive memory instead of 64 B from each
// of 16 rows that lie K elements apart.
__global__ void rd_pack_weights_kernel(const uint16_t *__restrict__ src, int N, int K, uint16_t *__restrict__ dst)
{
    const size_t tile = blockIdx.x;                              // (n/16) * (K/32) + k/32
    const int ks = (int)(tile % (size_t)(K >> 5)), nt = (int)(tile / (size_t)(K >> 5));
    const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
    const int n = nt * 16 + r16;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N) v = *reinterpret_cast<const uint4 *>(src + (size_t)n * K + ks * 32 + g * 8);
    *reinterpret_cast<uint4 *>(dst + (tile * 64 + lane) * 8) = v;
}

// Row tiles of rd_gemm_kernel's workgroups for a launch of `rows` rows.
int gemm_row_tiles(int rows) { return rows > 128 ? 16 : rows > 64 ? 8 : 4; }

// From 33 rows on any layer may run on rd_gemm_kernel, with fewer those of so many weights (few_rows_gemm).
constexpr int kGemmRows = 9, kGemmRows2 = 16;
constexpr size_t kGemmWeights = (size_t)96 << 20, kGemmWeights2 = (size_t)32 << 20;
bool gemm_layer(size_t rows, size_t weights)
{
    return rows > 32 || (rows >= kGemmRows2 && weights >= kGemmWeights2) || (rows >= kGemmRows && weights >= kGemmWeights);
}

struct Plan {
    size_t x_f32[3], x_bf[3], s_bf[2], logits, part_max, part_sum, part_cv, part_ci, row_score, row_tok, paths[2], cum[2], parent, tok, kpart, total;
};

Plan draft_plan(int B, int W, int L, int Dm, int V)
{
    Plan p;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
    const size_t M = (size_t)B * W, G = 2 * (size_t)Dm;
    for (int i = 0; i < 3; ++i) { p.x_f32[i] = take(M * G * 4); p.x_bf[i] = take(M * G * 2); }
    for (int i = 0; i < 2; ++i) p.s_bf[i] = take(M * Dm * 2);
    p.logits = take(M * (size_t)V * 4);
    const size_t chunks = ((size_t)V + kChunk - 1) / kChunk;
    p.part_max = take(M * chunks * 4);
    p.part_sum = take(M * chunks * 4);
    const size_t lists = chunks * 4 <= 64 ? chunks * 4 : chunks;   // wide beams keep four lists per chunk
    p.part_cv = take(M * lists * W * 4);
    p.part_ci = take(M * lists * W * 4);
    p.row_score = take(M * W * 4);
    p.row_tok = take(M * W * 4);
    for (int i = 0; i < 2; ++i) { p.paths[i] = take(M * L * 4); p.cum[i] = take(M * 4); }
    p.parent = take(M * 4 * (size_t)(L > 1 ? L - 1 : 1));       // parent rows of every drafted position
    p.tok = take(M * 4);
    p.kpart = take(gemm_layer(M, G * G) ? (size_t)kSplitMaxWgs * gemm_row_tiles((int)M) * kGemmCols * 1024 : 0);      // a launch's partial tiles
    p.total = off;
    return p;
}

int draft_check(const rd_draft_params *p, int B, int W, int L)
{
    if (!p || B <= 0 || W <= 0 || L <= 0) return RD_ERR_INVALID_ARG;
    if (p->Dm <= 0 || p->V <= 0 || p->n_mlp < 0) return RD_ERR_INVALID_ARG;
    if (p->Dm % 64 != 0) return RD_ERR_UNSUPPORTED;              // every wave's K share is whole 32-wide steps
    if (p->dtype != RD_BF16 && p->dtype != RD_F16) return RD_ERR_UNSUPPORTED;
    if (p->tiled != 0 && p->tiled != 1) return RD_ERR_INVALID_ARG;
    if (W > kMaxBeam || (long long)B * W > kMaxRows || W > p->V) return RD_ERR_UNSUPPORTED;
    if (p->V > kMaxVocab || L > RD_MAX_N) return RD_ERR_UNSUPPORTED;
    return RD_OK;
}

template <typename T, int MT, int NT, int NWV, int EPI>
void launch_linear_one(const LinArgs<T> &a, hipStream_t stream)
{
    if (a.tiled)
        hipLaunchKernelGGL((rd_linear_kernel<T, MT, NT, NWV, EPI, true>), dim3((a.N + 16 * NT - 1) / (16 * NT)), dim3(NWV * 64), 0, stream, a);
    else
        hipLaunchKernelGGL((rd_linear_kernel<T, MT, NT, NWV, EPI, false>), dim3((a.N + 16 * NT - 1) / (16 * NT)), dim3(NWV * 64), 0, stream, a);
}

// waves per workgroup: as many as give the launch about 16 waves per compute unit, as long as
// every wave gets whole k-steps inside one product and its registers allow that many residents
template <typename T, int MT, int NT, int EPI>
int launch_linear_nt(const LinArgs<T> &a, hipStream_t stream)
{
    const int ks1 = a.K1 / 32, ks2 = a.K2 / 32, wgs = (a.N + 16 * NT - 1) / (16 * NT);
    auto ok = [&](int nwv) {
        if (ks2 == 0) return ks1 % nwv == 0;
        return ks1 == ks2 && ks1 % (nwv / 2) == 0;
    };
    int nwv = 4;
    if (wgs * 4 < 4096 && ok(8)) nwv = 8;
    if (wgs * 8 < 4096 && ok(16)) nwv = 16;
    constexpr bool k16 = MT * NT <= 4 && MT + NT <= 5;          // 16 waves need <= 128 registers per lane
    if (nwv == 16) { if constexpr (k16) launch_linear_one<T, MT, NT, 16, EPI>(a, stream); else launch_linear_one<T, MT, NT, 8, EPI>(a, stream); }
    else if (nwv == 8) launch_linear_one<T, MT, NT, 8, EPI>(a, stream);
    else launch_linear_one<T, MT, NT, 4, EPI>(a, stream);
    return rd_check_launch();
}

// K split over as many workgroups per column group as bring the launch to about one per compute unit, with eight k-steps each
// at least.
int gemm_splits(int groups, int ks)
{
    const int splits = groups < kSplitMaxWgs ? kSplitMaxWgs / groups : 1, most = ks >= 8 ? ks / 8 : 1;
    return splits < most ? splits : most;
}

// Column tiles of a workgroup, up to 128 rows: 16, or as few as 13 where they split into more workgroups of the chip's 256, so that the
// tiles that one of them copies, k-steps times rows and columns, are fewer by a twelfth.  A workgroup computes 16 all the same, the matrix
// cores are not the bound.  13312 columns, K = 13312: 64 groups of 13 in four splits instead of 52 of 16 (256 workgroups instead of 208).
// us per call by 16 / so: hidden size 6656, 64 rows 1380 / 1368, 72 1504 / 1484, 96 1572 / 1542, 128 1682 / 1651, row-major 72 rows, 8000
// tokens 1140 / 1080; 7168, 64 rows 1581 / 1569; 5632, 72 rows 1217 / 1208; 8256, 64 rows 2023 / 1990.  Short walks gain nothing
// (72 rows, 1536 348 / 355), and where 16 are used they are a constant (as an argument 768, 72 rows take 1 % longer).
int gemm_columns(int rt, int N, int ks)
{
    int best = 16, least = 0;
    for (int cols = 16; cols >= 13; --cols) {
        const int groups = (N + 16 * cols - 1) / (16 * cols), splits = gemm_splits(groups, ks), steps = (ks + splits - 1) / splits;
        if (groups > kSplitMaxWgs || steps < 32) break;
        const int copied = steps * (rt + cols);
        if (cols == 16) least = copied - copied / 12;
        else if (copied < least || (best == 16 && copied == least)) { best = cols; least = copied; }
    }
    return best;
}

template <typename T, int RT, int CT, int WR, int WC, int EPI, bool TRIM>
int launch_gemm_cols(LinArgs<T> a, int cols, hipStream_t stream)
{
    const int groups = (a.N + 16 * cols - 1) / (16 * cols);
    a.cols = cols;
    a.ksplit = gemm_splits(groups, (a.K1 + a.K2) / 32);
    constexpr size_t smem = gemm_lds<RT, CT>();
    static std::atomic<unsigned long long> conf_t{0}, conf_r{0};
    const void *fn = a.tiled ? reinterpret_cast<const void *>(&rd_gemm_kernel<T, RT, CT, WR, WC, EPI, true, TRIM>)
                             : reinterpret_cast<const void *>(&rd_gemm_kernel<T, RT, CT, WR, WC, EPI, false, TRIM>);
    if (rd::ensure_dynamic_lds(fn, smem, a.tiled ? conf_t : conf_r) != RD_OK) return RD_ERR_HIP;
    const dim3 grid((groups * a.ksplit + 7) / 8 * 8);
    if (a.tiled) hipLaunchKernelGGL((rd_gemm_kernel<T, RT, CT, WR, WC, EPI, true, TRIM>), grid, dim3(WR * WC * 64), smem, stream, a);
    else hipLaunchKernelGGL((rd_gemm_kernel<T, RT, CT, WR, WC, EPI, false, TRIM>), grid, dim3(WR * WC * 64), smem, stream, a);
    if (a.ksplit == 1) return rd_check_launch();
    const int tiles = (a.M + 15) / 16 * ((a.N + 15) / 16);
    hipLaunchKernelGGL((rd_linear_finish_kernel<T, RT, CT, EPI, TRIM>), dim3((tiles + 3) / 4), dim3(256), 0, stream, a);
    return rd_check_launch();
}

template <typename T, int RT, int CT, int WR, int WC, int EPI>
int launch_gemm(const LinArgs<T> &a, hipStream_t stream)
{
    if constexpr (gemm_trims<RT, CT>()) {
        const int cols = gemm_columns(RT, a.N, (a.K1 + a.K2) / 32);
        if (cols < CT) return launch_gemm_cols<T, RT, CT, WR, WC, EPI, true>(a, cols, stream);
    }
    return launch_gemm_cols<T, RT, CT, WR, WC, EPI, false>(a, CT, stream);
}

// The output layer at 9 rows and more per launch, wide enough to cover half the chip with 128-column
// workgroups: waves split the columns, activations staged in LDS (rd_head_rows_kernel).  Measured per call
// at a hidden size of 4096 and 32000 tokens against the K-split kernels: 16 rows 832 -> 766 us, 32 rows
// 919 -> 835, 64 rows 1007 -> 965, 128 rows 1400 -> 1173 (8 rows 725 -> 730; rd_stream_kernel takes 627).
template <typename T, int MT, int EPI>
bool launch_head_rows(const LinArgs<T> &a, hipStream_t stream, int *status)
{
    if constexpr (MT >= 1 && EPI == EPI_HEAD) {
        static const int on = rd::env_int("RD_DRAFT_HEAD_ROWS", 1);    // 0: the K-split kernel (for comparisons)
        if (!on || a.K2 != 0 || a.map1 != nullptr || a.K1 % kRowsKC != 0 || a.N < 128 * 128) return false;
        if (a.M <= 8) return false;                                    // up to 8 rows the kernels that split K are faster
        constexpr size_t smem = 2 * (size_t)MT * 16 * kRowsStride;
        static std::atomic<unsigned long long> conf_t{0}, conf_r{0};
        const void *fn = a.tiled ? reinterpret_cast<const void *>(&rd_head_rows_kernel<T, MT, true>)
                                 : reinterpret_cast<const void *>(&rd_head_rows_kernel<T, MT, false>);
        if (rd::ensure_dynamic_lds(fn, smem, a.tiled ? conf_t : conf_r) != RD_OK) { *status = RD_ERR_HIP; return true; }
        const dim3 grid((a.N + 127) / 128);
        if (a.tiled) hipLaunchKernelGGL((rd_head_rows_kernel<T, MT, true>), grid, dim3(512), smem, stream, a);
        else hipLaunchKernelGGL((rd_head_rows_kernel<T, MT, false>), grid, dim3(512), smem, stream, a);
        *status = rd_check_launch();
        return true;
    } else {
        return false;
    }
}

// Up to 32 rows without the column-split kernel: column tiles per workgroup, the most that still leave about one workgroup per
// compute unit (the activation re-reads are MT : NT of the weight bytes, and measured they cost as much as the
// weights' own stream; halving the workgroups below the number of compute units costs more)
template <typename T, int MT, int EPI>
int launch_linear_mt(const LinArgs<T> &a, hipStream_t stream)
{
    if constexpr (MT == 2) {
        if (a.N >= 240 * 128) return launch_linear_nt<T, MT, 8, EPI>(a, stream);
        if (a.N >= 256 * 32) return launch_linear_nt<T, MT, 2, EPI>(a, stream);
    }
    return launch_linear_nt<T, MT, 1, EPI>(a, stream);
}

// Which kernel runs a layer.  rd_gemm_kernel, 256 rows at a time, from 33 rows on (with fewer: few_rows_gemm), but for the output
// layer up to 128 rows, which rd_head_rows_kernel runs without splitting K (us per call at a hidden size of 4096, 64 rows 877 /
// 861, 128 rows 1044 / 1012), and for layers of up to 8 Mi weights and 64 rows, which take less time than a second launch costs
// (rd_linear_kernel; 40 rows, us per call by hidden size, the limit at none / 1 / 4 / 8 / 16 Mi: 512 112 / 98 / 89 / 89 / 89,
// 1024 121 / 121 / 114 / 107 / 107; 64 rows, 1536 140 / 140 / 140 / 139 / 143).  65 to 128 column groups of few k-steps take
// workgroups of half as many columns, which need no split (80 rows, hidden size 704, 20445 tokens 154 -> 151, 128 rows 168 -> 160;
// with many k-steps they take longer: hidden size 8256 689 -> 812).
constexpr size_t kSmallLayer = 8u << 20;

// 9 to 32 rows: rd_linear_kernel reads every activation once per 16 columns and fills the chip in whole rounds of workgroups
// only at some sizes, rd_gemm_kernel pays a second launch.  us per call of four MLP layers at 8 / 12 / 16 / 24 / 32 rows, hidden
// size 2048 by the former 50 / 51 / 52 / 63 / 69, by the latter 75 / 75 / 75 / 78 / 79; 3072 108 / 118 / 133 / 162 / 183 and
// 113 / 112 / 112 / 116 / 117; 4096 135 / 146 / 162 / 171 / 184 and 162 / 161 / 161 / 167 / 168; 5120 210 / 231 / 258 / 320 / 355
// and 204 / 203 / 205 / 210 / 213; 6656 336 / 376 / 421 / 411 / 458 and 302 / 301 / 304 / 312 / 318.
// Where rd_linear_kernel's workgroups of 16 columns are whole rounds of 256 it stays up to 24 rows while the activations, read
// with every weight, cost less than the second launch: rows times weights up to 1.5 Gi.  us per call by it / by rd_gemm_kernel:
// hidden size 4096, 16 and 24 rows 735 / 743 and 756 / 760; three MLP layers and two positions at 9 / 12 / 16 / 24 rows, 6144
// 459 / 501 / 554 / 660 and 478 / 484 / 491 / 514, 8192 776 / 833 / 907 / 929 and 771 / 778 / 786 / 808, 10240 1144 / 1259 / 1417 / 1536
// and 1081 / 1088 / 1100 / 1136.
bool few_rows_gemm(int rows, int N, int K)
{
    const size_t weights = (size_t)N * K;
    if (rows <= 24 && N % (16 * 256) == 0 && rows * weights <= (size_t)1536 << 20) return false;
    return gemm_layer(rows, weights);
}

// Up to 8 rows, where the layer is more than kSmallLayer and every wave has a few units of K: below that the rings only add to
// the launch (hidden size 512, 8000 tokens 99.6 us per call by rd_linear_kernel, 101.8 by this; 1024, 32000 177.4 and 178.0 with
// all layers, the output layer alone is above the line).
bool stream_layer(int rows, int N, int K) { return rows <= kStreamRows && (size_t)N * K > kSmallLayer && K >= 2048; }

template <typename T, int EPI>
int launch_stream(const LinArgs<T> &a, hipStream_t stream)
{
    static std::atomic<unsigned long long> conf_t{0}, conf_r{0};
    const void *fn = a.tiled ? reinterpret_cast<const void *>(&rd_stream_kernel<T, EPI, true>)
                             : reinterpret_cast<const void *>(&rd_stream_kernel<T, EPI, false>);
    if (rd::ensure_dynamic_lds(fn, kStreamLds, a.tiled ? conf_t : conf_r) != RD_OK) return RD_ERR_HIP;
    const dim3 grid((a.N + 15) / 16);
    if (a.tiled) hipLaunchKernelGGL((rd_stream_kernel<T, EPI, true>), grid, dim3(kStreamWaves * 64), kStreamLds, stream, a);
    else hipLaunchKernelGGL((rd_stream_kernel<T, EPI, false>), grid, dim3(kStreamWaves * 64), kStreamLds, stream, a);
    return rd_check_launch();
}

// Layers of up to 64 rows take workgroups of half as many columns also where half the splits of K then fill the chip, three or more:
// half the partial sums to write and read.  With two the activations, read twice as often, cost more.  us per call, 64 rows of hidden
// size 4096 797 / 780, 3072 615 / 597, 5120 999 / 995, 36 rows of 1536 257 / 250; two splits, 50 rows of 7680 1685 / 1731; a chip
// filled to four fifths, 64 rows of 6656 1440 / 1509, 4608 929 / 940.
bool gemm_halves(int N)
{
    const int groups = (N + 127) / 128, splits = kSplitMaxWgs / groups;
    return splits >= 3 && groups * splits >= kSplitMaxWgs * 15 / 16;
}

template <typename T, int EPI>
int launch_linear(const LinArgs<T> &all, hipStream_t stream)
{
    for (int m0 = 0, rows; m0 < all.M; m0 += rows) {
        rows = all.M - m0 < 256 ? all.M - m0 : 256;
        LinArgs<T> a = all;
        a.m0 = m0;
        a.M = rows;
        const int mt = (rows + 15) / 16;
        int st = RD_OK;
        bool done = false;
        if (stream_layer(rows, a.N, a.K1 + a.K2)) {
            st = launch_stream<T, EPI>(a, stream);
            done = true;
        } else if constexpr (EPI == EPI_HEAD) {
            if (mt <= 1) done = launch_head_rows<T, 1, EPI>(a, stream, &st);
            else if (mt <= 2) done = launch_head_rows<T, 2, EPI>(a, stream, &st);
            else if (mt <= 4) done = launch_head_rows<T, 4, EPI>(a, stream, &st);
            else if (mt <= 8) done = launch_head_rows<T, 8, EPI>(a, stream, &st);
        }
        if (!done && mt > 2 && mt <= 4 && (size_t)a.N * (a.K1 + a.K2) <= kSmallLayer) {
            st = launch_linear_nt<T, 4, 1, EPI>(a, stream);
            done = true;
        }
        if (!done) {
            if (all.M > 32 || (EPI != EPI_HEAD && few_rows_gemm(rows, a.N, a.K1 + a.K2))) {
                const int rt = gemm_row_tiles(rows), groups = (a.N + 16 * kGemmCols - 1) / (16 * kGemmCols);
                const bool narrow = (groups > 64 && groups <= 128 && a.K1 + a.K2 <= 4096) || (rt == 4 && gemm_halves(a.N));
                if (rt == 16) st = launch_gemm<T, 16, 16, 2, 4, EPI>(a, stream);
                else if (rt == 8) st = narrow ? launch_gemm<T, 8, 8, 2, 4, EPI>(a, stream) : launch_gemm<T, 8, 16, 2, 4, EPI>(a, stream);
                else st = narrow ? launch_gemm<T, 4, 8, 2, 4, EPI>(a, stream) : launch_gemm<T, 4, 16, 1, 8, EPI>(a, stream);
            } else if (mt <= 1) {
                st = launch_linear_mt<T, 1, EPI>(a, stream);
            } else {
                st = launch_linear_mt<T, 2, EPI>(a, stream);
            }
        }
        if (st != RD_OK) return st;
    }
    return RD_OK;
}

// The whole call for one storage type (launches only; arguments already checked).
template <typename E>
int draft_run(const rd_draft_params *p, const void *h, const int32_t *last_token, int B, int W, int L,
              int32_t *beams, float *beam_logp, float *step_logits, int32_t *step_row,
              void *workspace, size_t workspace_bytes, void *stream)
{
    const Plan plan = draft_plan(B, W, L, p->Dm, p->V);
    if (!workspace || !rd_aligned(workspace, 256) || workspace_bytes < plan.total) return RD_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    const int Dm = p->Dm, G = 2 * Dm, V = p->V, M = B * W, T = L - 1;
    float *x_f32[3];
    E *x_bf[3], *s_bf[2];
    for (int i = 0; i < 3; ++i) { x_f32[i] = reinterpret_cast<float *>(ws + plan.x_f32[i]); x_bf[i] = reinterpret_cast<E *>(ws + plan.x_bf[i]); }
    for (int i = 0; i < 2; ++i) s_bf[i] = reinterpret_cast<E *>(ws + plan.s_bf[i]);
    float *logits = reinterpret_cast<float *>(ws + plan.logits);
    float *part_max = reinterpret_cast<float *>(ws + plan.part_max), *part_sum = reinterpret_cast<float *>(ws + plan.part_sum);
    float *part_cv = reinterpret_cast<float *>(ws + plan.part_cv);
    int32_t *part_ci = reinterpret_cast<int32_t *>(ws + plan.part_ci);
    float *row_score = reinterpret_cast<float *>(ws + plan.row_score);
    int32_t *row_tok = reinterpret_cast<int32_t *>(ws + plan.row_tok);
    const int chunks = (V + kChunk - 1) / kChunk;
    int32_t *paths[2] = {reinterpret_cast<int32_t *>(ws + plan.paths[0]), reinterpret_cast<int32_t *>(ws + plan.paths[1])};
    float *cum[2] = {reinterpret_cast<float *>(ws + plan.cum[0]), reinterpret_cast<float *>(ws + plan.cum[1])};
    int32_t *parent = reinterpret_cast<int32_t *>(ws + plan.parent), *tok = reinterpret_cast<int32_t *>(ws + plan.tok);
    float *kpart = reinterpret_cast<float *>(ws + plan.kpart);
    const E *emb = static_cast<const E *>(p->emb);

    hipLaunchKernelGGL(rd_draft_init_kernel<E>, dim3(M, (Dm + 2047) / 2048), dim3(256), 0, s, emb, static_cast<const E *>(h), last_token,
                       W, L, Dm, V, x_f32[0], x_bf[0], s_bf[0], paths[0], cum[0]);
    if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
    if (T == 0) {                                   // nothing to draft: the candidates are the LLM's token alone
        hipLaunchKernelGGL(rd_draft_init_kernel<E>, dim3(M, (Dm + 2047) / 2048), dim3(256), 0, s, emb, static_cast<const E *>(h), last_token,
                           W, L, Dm, V, x_f32[0], x_bf[0], s_bf[0], beams, beam_logp);
        return rd_check_launch();
    }
    // the h half of X0 must survive the MLP ping-pong: layers write X1 and X2 only
    int si = 0;                                     // state buffer holding s_t of the live candidates
    for (int t = 1; t <= T; ++t) {
        const int cur = (t - 1) & 1, nxt = t & 1;
        if (t > 1) {                                // s_t = f(U s_{t-1}[parent] + W e(token) + b) -> X0[:, :Dm]
            LinArgs<E> a = {};
            a.w1 = static_cast<const E *>(p->rnn_u); a.x1 = s_bf[si]; a.map1 = parent + (size_t)(t - 2) * M; a.ldx1 = Dm; a.K1 = Dm;
            a.w2 = static_cast<const E *>(p->rnn_w); a.x2 = emb; a.map2 = tok; a.ldx2 = Dm; a.K2 = Dm;
            a.bias = p->rnn_b; a.M = M; a.N = Dm; a.mstride = 1; a.tiled = p->tiled;
            a.y_f32 = x_f32[0]; a.y_bf = x_bf[0]; a.s_bf = s_bf[si ^ 1]; a.ldy = G; a.kpart = kpart;
            if (launch_linear<E, EPI_RNN>(a, s) != RD_OK) return RD_ERR_HIP;
            si ^= 1;
        }
        // at the first position the W rows of a sequence are one and the same state: compute row b*W only
        const int rows = t == 1 ? B : M, mstride = t == 1 ? W : 1;
        int in = 0;
        for (int k = 0; k < p->n_mlp; ++k) {        // x <- x + f(A_k x + c_k)
            const int out = in == 1 ? 2 : 1;
            LinArgs<E> a = {};
            a.w1 = static_cast<const E *>(p->mlp_w) + (size_t)k * G * G; a.x1 = x_bf[in]; a.ldx1 = G; a.K1 = G;
            a.bias = p->mlp_b + (size_t)k * G; a.M = rows; a.N = G; a.mstride = mstride; a.tiled = p->tiled;
            a.y_f32 = x_f32[out]; a.y_bf = x_bf[out]; a.res = x_f32[in]; a.ldy = G; a.kpart = kpart;
            if (launch_linear<E, EPI_MLP>(a, s) != RD_OK) return RD_ERR_HIP;
            in = out;
        }
        {                                           // logits
            LinArgs<E> a = {};
            a.w1 = static_cast<const E *>(p->head_w); a.x1 = x_bf[in]; a.ldx1 = G; a.K1 = G;
            if (step_logits) logits = step_logits + (size_t)(t - 1) * M * V;   // every position keeps its matrix
            a.M = rows; a.N = V; a.mstride = mstride; a.tiled = p->tiled; a.y_f32 = logits; a.ldy = V; a.kpart = kpart;
            if (launch_linear<E, EPI_HEAD>(a, s) != RD_OK) return RD_ERR_HIP;
        }
        // with many candidates (and while four lists per chunk fit the row pass's 64 lanes) the chunk pass
        // leaves its four waves' lists unmerged
        const bool few = W <= kFewBeam;
        const int lpc = (!few && chunks * 4 <= 64) ? 4 : 1;
        if (few)
            hipLaunchKernelGGL(rd_topw_few_kernel, dim3(chunks, rows), dim3(kChunkThreads), 0, s, logits, V, W, chunks, mstride,
                               part_max, part_sum, part_cv, part_ci);
        else
            hipLaunchKernelGGL(rd_topw_chunk_kernel, dim3(chunks, rows), dim3(kChunkThreads), 0, s, logits, V, W, chunks, mstride, lpc,
                               part_max, part_sum, part_cv, part_ci);
        if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
        const bool last = t == T;
        const bool wide = W > kNarrowBeam;
        const int live = t == 1 ? 1 : W;
        if (few_lists(W, chunks)) {
            hipLaunchKernelGGL(rd_row_beam_kernel, dim3(B), dim3(kSelThreads), 0, s, part_max, part_sum, part_cv, part_ci, chunks,
                               cum[cur], V, W, L, t, live, paths[cur], paths[nxt], cum[nxt], parent + (size_t)(t - 1) * M, tok,
                               last ? beams : nullptr, last ? beam_logp : nullptr);
            if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
            continue;
        }
#define RD_ROW_LAUNCH(LPR, WMAX, grid)                                                                                   \
        hipLaunchKernelGGL((rd_topw_row_kernel<LPR, WMAX>), dim3(grid), dim3(kSelThreads), 0, s, part_max, part_sum, part_cv, part_ci, \
                           chunks, lpc, cum[cur], W, rows, mstride, row_score, row_tok)
        if (chunks * lpc <= 8) {
            if (wide) RD_ROW_LAUNCH(8, kMaxBeam, (rows + 7) / 8); else RD_ROW_LAUNCH(8, kNarrowBeam, (rows + 7) / 8);
        } else {
            if (wide) RD_ROW_LAUNCH(64, kMaxBeam, rows); else RD_ROW_LAUNCH(64, kNarrowBeam, rows);
        }
#undef RD_ROW_LAUNCH
        if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
        if (wide) {
            static std::atomic<unsigned long long> configured{0};
            if (rd::ensure_dynamic_lds(reinterpret_cast<const void *>(&rd_beam_step_kernel<true>), (size_t)kMaxBeam * kMaxBeam * 8,
                                       configured) != RD_OK)
                return RD_ERR_HIP;
            hipLaunchKernelGGL(rd_beam_step_kernel<true>, dim3(B), dim3(kSelThreads), (size_t)live * W * 8, s, row_score, row_tok, V, W, L, t,
                               live, paths[cur], paths[nxt], cum[nxt], parent + (size_t)(t - 1) * M, tok,
                               last ? beams : nullptr, last ? beam_logp : nullptr);
        } else {
            hipLaunchKernelGGL(rd_beam_step_kernel<false>, dim3(B), dim3(kSelThreads), 0, s, row_score, row_tok, V, W, L, t,
                               live, paths[cur], paths[nxt], cum[nxt], parent + (size_t)(t - 1) * M, tok,
                               last ? beams : nullptr, last ? beam_logp : nullptr);
        }
        if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
    }
    if (step_row) {
        hipLaunchKernelGGL(rd_draft_rows_kernel, dim3((M + 255) / 256), dim3(256), 0, s, parent, M, W, T, step_row);
        if (rd_check_launch() != RD_OK) return RD_ERR_HIP;
    }
    return RD_OK;
}

}  // namespace

extern "C" size_t rd_draft_workspace(int B, int W, int L, int Dm, int V)
{
    rd_draft_params p = {};
    p.Dm = Dm; p.V = V; p.dtype = RD_BF16;
    if (draft_check(&p, B, W, L) != RD_OK) return 0;
    return draft_plan(B, W, L, Dm, V).total;
}

extern "C" int rd_draft(const rd_draft_params *p, const void *h, const int32_t *last_token,
                        int B, int W, int L, int32_t *beams, float *beam_logp,
                        float *step_logits, int32_t *step_row,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    const int st = draft_check(p, B, W, L);
    if (st != RD_OK) return st;
    if (!p->emb || !p->rnn_u || !p->rnn_w || !p->rnn_b || !p->head_w || (p->n_mlp > 0 && (!p->mlp_w || !p->mlp_b)))
        return RD_ERR_INVALID_ARG;
    if (!h || !last_token || !beams || !beam_logp) return RD_ERR_INVALID_ARG;
    if ((step_logits == nullptr) != (step_row == nullptr) || !rd_aligned(step_logits, 16)) return RD_ERR_INVALID_ARG;
    if (!rd_aligned(p->emb, 16) || !rd_aligned(p->rnn_u, 16) || !rd_aligned(p->rnn_w, 16) || !rd_aligned(p->mlp_w, 16) ||
        !rd_aligned(p->head_w, 16) || !rd_aligned(h, 16))
        return RD_ERR_INVALID_ARG;
    if (p->dtype == RD_F16)
        return draft_run<_Float16>(p, h, last_token, B, W, L, beams, beam_logp, step_logits, step_row, workspace, workspace_bytes, stream);
    return draft_run<__bf16>(p, h, last_token, B, W, L, beams, beam_logp, step_logits, step_row, workspace, workspace_bytes, stream);
}

extern "C" size_t rd_draft_packed_elems(int N, int K)
{
    if (N <= 0 || K <= 0 || K % 32 != 0) return 0;
    return (size_t)((N + 15) / 16 * 16) * (size_t)K;
}

extern "C" int rd_draft_pack_weights(const void *src, int N, int K, void *dst, void *stream)
{
    if (!src || !dst || N <= 0 || K <= 0) return RD_ERR_INVALID_ARG;
    if (K % 32 != 0) return RD_ERR_UNSUPPORTED;
    if (!rd_aligned(src, 16) || !rd_aligned(dst, 16)) return RD_ERR_INVALID_ARG;
    const size_t tiles = (size_t)((N + 15) / 16) * (size_t)(K / 32);
    if (tiles > 0x7fffffffull) return RD_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(rd_pack_weights_kernel, dim3((unsigned)tiles), dim3(64), 0, (hipStream_t)stream,
                       static_cast<const uint16_t *>(src), N, K, static_cast<uint16_t *>(dst));
    return rd_check_launch();
}
