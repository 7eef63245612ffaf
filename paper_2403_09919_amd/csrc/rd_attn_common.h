// Pieces shared by the tree-attention kernels: the launch plans and the exchange in which the last
// workgroup of a (sequence, head) to finish learns that it is.
//
// Work decomposition (flash-decoding style).  The keys a packed row may see are the context keys
// 0..ctx_len-1 plus the packed keys allowed by its mask row (Sec. 3.3).  The keys of a (sequence, head) are cut
// into ranges, one workgroup each; it computes, for all packed rows (or a group of them) at once, a partial softmax
// state (running max m, sum l, unnormalised output O).  A head with one range is written out directly; else
// the state goes to the workspace and the workgroup that finishes last for that head -- found with a device-scope
// counter -- merges the partials, normalises and writes the output, so the whole operation is a single launch.
#pragma once
#include "rd_internal.h"
#include <math.h>

namespace rd {

constexpr int kAttnThreads = 256;
constexpr int kBlockKeys = 128;   // keys handled per workgroup iteration

struct AttnPlan {
    int waves;         // matrix-core kernel: waves per workgroup (4 or 8); a block is 32*waves keys
    int S;             // workgroups per (sequence, head); fp32 kernel: context ranges, one more workgroup takes the packed keys
    int rows_pad;      // packed rows padded to a multiple of 16 (fp32 kernel's partial layout)
    int rg_tiles;      // matrix-core kernel: 16-row tiles of packed rows per workgroup (a row group)
    int n_rg;          // ... row groups per (sequence, head); 1 unless N is large
    size_t counters_bytes;
    size_t total_bytes;
};

// Plan of the matrix-core kernel (rd_tree_attn_mfma.h), for contexts of up to Cmax keys: waves per workgroup, rows
// per workgroup and workgroups per head, from an estimate of the launch time.  Lengths are upper bounds and the
// packed rows are not known at all here (distinct prefixes are taken to be 0.6 of the candidates' tokens); the kernel
// deals its tiles to the workgroups from the lengths it finds.  Measured on MI355X, us, at D = 128 (D = 64: blocks take 0.6 of it):
//   * a workgroup is 1.0 (eight waves) or 1.2 (four) plus 2.0 + 0.5 r or 1.15 + 0.3 r per block, r = row tiles with
//     packed rows; at five row tiles K comes in operand order, 0.3 more per block of eight waves;
//   * one eight-wave workgroup fills a compute unit, two of four waves do; more start as those retire;
//   * the workgroups that run at one time share 5.0 (eight waves) or 5.25 TB/s, a compute unit gets 28 GB/s at most,
//     and one with two workgroups takes twice as long as one with one (the rest of the chip then idles, which leaves
//     the others more: half of that is counted); latency and bandwidth overlap in part (root of the sum of squares);
//   * more than one range per head adds a merge: 1.5, and the partial results written and read back, the reading by
//     one compute unit at 50 GB/s.
// Beams of more than 80 packed rows are cut into row groups, as equal as whole tiles allow; every group walks the
// head's keys, and workgroups of groups that turn out empty go to the others.
static inline AttnPlan attn_plan_make(int B, int H, int N, int D, int Cmax)
{
    constexpr int kMaxTilesPerGroup = 5, kWideTilesPerGroup = 4;    // as instantiated
    const long long BH = (long long)B * H;
    const int nq_all = (N + 15) / 16;
    const double rows = 0.6 * N, scale = D == 128 ? 1.0 : 0.6;
    const int tiles = (Cmax + 31) / 32 + ((int)rows + 31) / 32;
    static const int waves_env = env_int("RD_ATTN_WAVES", 0), forced = env_int("RD_ATTN_SPLITS", 0);
    AttnPlan best = {};
    double best_T = 1e30;
    for (int waves = 8; waves >= 4; waves -= 4) {
        if (waves_env && waves != waves_env) continue;
        int n_rg = (nq_all + kMaxTilesPerGroup - 1) / kMaxTilesPerGroup;
        const int nq = N > 32 * waves ? kWideTilesPerGroup : (nq_all + n_rg - 1) / n_rg;
        n_rg = (nq_all + nq - 1) / nq;
        int n_act = (int)((rows + 16 * nq - 1) / (16 * nq));
        n_act = n_act < 1 ? 1 : n_act;
        double r = n_act > 1 ? nq : (rows + 15) / 16;
        r = r < 1 ? 1 : (r > nq ? nq : r);
        const int nblk = tiles > waves ? (tiles + waves - 1) / waves : 1;
        const double t_blk = scale * (waves == 8 ? 2.0 + 0.5 * r + (nq > 4 ? 0.3 : 0.0) : 1.15 + 0.3 * r);
        const double t_wg = waves == 8 ? 1.0 : 1.2, rate = waves == 8 ? 5.0e6 : 5.25e6;
        const long long slots = waves == 8 ? 256 : 512;
        const double part = r * 16 * (2 + D) * sizeof(float);
        for (int S = n_rg; S <= 64 * n_rg && S <= nblk * n_rg; ++S) {
            const int ranges = S / n_act, per = (nblk + ranges - 1) / ranges, n_part = (nblk + per - 1) / per;
            const double t_lat = t_wg + per * t_blk, bytes = (double)(per * waves < tiles ? per * waves : tiles) * 32 * D * 4 / n_act;
            const long long wgs = (BH + 7) / 8 * 8 * S, full = wgs / slots, rest = wgs % slots;
            auto round = [&](long long n) {
                const long long per_cu = (n + 255) / 256;
                const double sharing = ((n < 256 ? n : 256) + (double)n / per_cu) / 2;
                const double t_bw = per_cu * bytes / (rate / sharing < 28e3 ? rate / sharing : 28e3);
                return sqrt(t_lat * t_lat + t_bw * t_bw);
            };
            double T = full * round(slots) + (rest ? round(rest) : 0.0);
            if (n_part > 1) T += 1.5 + n_part * part / 50e3 + 2.0 * (double)BH * n_act * n_part * part / 4e6;
            const bool take = forced > 0 ? S == (forced < n_rg ? n_rg : (forced < nblk * n_rg ? forced : nblk * n_rg)) : T < best_T * (1 - 1e-9);
            if (take) {
                best_T = T;
                best.waves = waves;
                best.S = S;
                best.rg_tiles = nq;
                best.n_rg = n_rg;
                best.counters_bytes = ((size_t)BH * n_rg * sizeof(unsigned long long) + 255) / 256 * 256;
                best.total_bytes = best.counters_bytes + (S > 1 ? (size_t)BH * S * (size_t)(nq * 16 * (2 + D)) * sizeof(float) : 0);
            }
        }
    }
    best.rows_pad = nq_all * 16;
    return best;
}

// The search takes up to some microseconds; a program calls with the same few shapes, so each thread keeps its last plan.
static inline AttnPlan attn_plan(int B, int H, int N, int D, int Cmax)
{
    static thread_local int key[5] = {0, 0, 0, 0, -1};
    static thread_local AttnPlan plan;
    if (key[0] != B || key[1] != H || key[2] != N || key[3] != D || key[4] != Cmax) {
        plan = attn_plan_make(B, H, N, D, Cmax);
        key[0] = B; key[1] = H; key[2] = N; key[3] = D; key[4] = Cmax;
    }
    return plan;
}

// Plan of the fp32 kernel: context ranges per head, estimated as above from what it does (27 GB/s per compute unit).
static inline AttnPlan attn_plan_f32(int B, int H, int N, int D, int Cmax)
{
    AttnPlan p = {};
    const long long BH = (long long)B * H;
    const int nblk = (Cmax + kBlockKeys - 1) / kBlockKeys, rows_pad = (N + 15) / 16 * 16;
    const double blk_bytes = 2.0 * kBlockKeys * D * sizeof(float), t_blk = blk_bytes / 27e9;
    const double t_hbm = (double)BH * nblk * blk_bytes / 5.5e12;
    const double part_bytes = (double)rows_pad * (2 + D) * sizeof(float);
    int best_S = 1;
    double best_T = 1e30;
    for (int S = 1; S <= nblk && S <= 64; ++S) {
        const int per = (nblk + S - 1) / S;
        const long long rounds = (BH * S + 255) / 256;
        double T = (double)rounds * per * t_blk;
        if (T < t_hbm) T = t_hbm;
        T += 3e-6 + 2.0 * (double)BH * (S + 1) * part_bytes / 4e12;
        if (T < best_T * (1.0 - 1e-9)) { best_T = T; best_S = S; }
    }
    p.waves = 4;
    p.S = best_S;
    p.rows_pad = rows_pad;
    p.rg_tiles = 1;
    p.n_rg = 1;
    p.counters_bytes = ((size_t)BH * sizeof(unsigned long long) + 255) / 256 * 256;
    p.total_bytes = p.counters_bytes + (size_t)BH * (p.S + 1) * (size_t)rows_pad * (2 + D) * sizeof(float);
    return p;
}

struct AttnArgs {
    const void *q, *k_cache, *v_cache, *k_new, *v_new;
    const int32_t *ctx_len, *n_packed;
    const int32_t *block_table;   // paged cache only: [B, max_pages] page of keys [j*page_size, (j+1)*page_size)
    int page_size, max_pages, n_pages;
    const uint64_t *mask_bits;
    void *out;
    unsigned long long *counters;
    float *partials;
    int B, H, N, Cmax, S, words, rows_pad;
    int n_rg;      // row groups per (sequence, head) (matrix-core kernel; each is NQ*16 rows of the template)
    float scale_log2e;
    // rotary embedding fused into the call (rd_tree_attn_rope); unused (null) otherwise
    const int32_t *position_ids;   // [B, N]
    const float *cos_tab, *sin_tab;   // [max_pos, D/2]
    int max_pos;
    void *k_rot;                   // [B,H,N,D] rotated packed keys (output), or null
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// Context key range [k_begin, k_end) of split s out of S for a context of C keys: whole
// blocks of block_keys keys, spread as evenly as whole blocks allow.
__device__ __forceinline__ void ctx_range(int C, int S, int s, int block_keys, int *k_begin, int *k_end)
{
    const int nblk = (C + block_keys - 1) / block_keys;
    const int per = (nblk + S - 1) / S;
    const int kb = s * per * block_keys;
    *k_begin = kb < C ? kb : C;
    const int ke = kb + per * block_keys;
    *k_end = ke < C ? ke : C;
}

__device__ __forceinline__ void store_out4(float *dst, float a, float b, float c, float d)
{
    *reinterpret_cast<float4 *>(dst) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void store_out4(__bf16 *dst, float a, float b, float c, float d)
{
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    bf16x4 v;
    v[0] = (__bf16)a; v[1] = (__bf16)b; v[2] = (__bf16)c; v[3] = (__bf16)d;   // round to nearest even
    *reinterpret_cast<bf16x4 *>(dst) = v;
}

__device__ __forceinline__ void store_out4(_Float16 *dst, float a, float b, float c, float d)
{
    typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
    f16x4 v;
    v[0] = (_Float16)a; v[1] = (_Float16)b; v[2] = (_Float16)c; v[3] = (_Float16)d;   // round to nearest even
    *reinterpret_cast<f16x4 *>(dst) = v;
}

// XCD this workgroup runs on (hardware register XCC_ID).
__device__ __forceinline__ uint32_t xcc_id() { return __builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xfu; }

enum { kNotLast = 0, kLastClean = 1, kLastMixed = 2 };

// Signals that this workgroup's partial is stored (with st_dev*); tells every thread of the
// workgroup whether it arrived last among `expected` for this (sequence, head).  The last arriver
// also learns whether every contributor ran on its own XCD (kLastClean: the partials are then
// current in its L2, which is coherent within an XCD) or not (kLastMixed: it must read them with
// ld_dev*, past its L2, which may still hold an older call's lines).  No assumption is made about
// which XCD a workgroup lands on: the 64-bit word collects, beside the count (bits 0-15), the sum
// (bits 16-31) and the sum of squares (bits 32-63) of the contributors' XCD numbers, and n values
// are all equal to x exactly if their sum is n*x and their sum of squares n*x*x.
__device__ __forceinline__ int arrive_is_last(unsigned long long *counter, uint32_t expected)
{
    __shared__ uint32_t s_last;
    wait_dev_stores();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // waits until this thread's stores are acknowledged
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long x = xcc_id();
        const unsigned long long add = 1ull | (x << 16) | ((x * x) << 32);
        const unsigned long long now = __hip_atomic_fetch_add(counter, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
        const unsigned long long n = now & 0xffffull;
        const bool same = ((now >> 16) & 0xffffull) == n * x && (now >> 32) == n * x * x;
        s_last = (n == expected) ? (same ? kLastClean : kLastMixed) : kNotLast;
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // later loads stay after the counter update
    return (int)s_last;
}

// Merge of the S+1 partial softmax states of one (sequence, head) and final store:
// out[p] = sum_s 2^(m_s - M) O_s[p] / sum_s 2^(m_s - M) l_s[p] with M = max_s m_s (scores
// are kept in log2 units).  Rows p >= P are written as zero.  Run by one workgroup.
template <int D, typename OutT>
__device__ __forceinline__ void combine_partials(const float *part /* first partial of this head */,
                                                 int n_part, size_t partial_floats, int rows_pad,
                                                 int P, int N, OutT *out /* [N][D] of this head */)
{
    constexpr int kVecPerRow = D / 4;
    constexpr int kRowsPerPass = kAttnThreads / kVecPerRow;
    const int tid = threadIdx.x;
    const int v = tid % kVecPerRow;
    for (int p = tid / kVecPerRow; p < N; p += kRowsPerPass) {
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
        if (p < P) {
            float M = -INFINITY;
            for (int s = 0; s < n_part; ++s) M = fmaxf(M, ld_dev(part + s * partial_floats + p));
            float denom = 0.f;
            for (int s = 0; s < n_part; ++s) {
                const float *ps = part + s * partial_floats;
                const float m = ld_dev(ps + p);
                if (m == -INFINITY) continue;          // that range held no visible key for row p
                const float w = __builtin_amdgcn_exp2f(m - M);
                denom += w * ld_dev(ps + rows_pad + p);
                const float *po = ps + 2 * rows_pad + (size_t)p * D + 4 * v;
                const float2 o01 = ld_dev2(po), o23 = ld_dev2(po + 2);
                a0 += w * o01.x; a1 += w * o01.y; a2 += w * o23.x; a3 += w * o23.y;
            }
            const float inv = 1.0f / denom;
            a0 *= inv; a1 *= inv; a2 *= inv; a3 *= inv;
        }
        store_out4(out + (size_t)p * D + 4 * v, a0, a1, a2, a3);
    }
}

}  // namespace rd
