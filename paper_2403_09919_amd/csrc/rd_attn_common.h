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

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kOneStep = 64;     // sequences that the lanes of a wave hold one by one

struct AttnPlan {
    int waves;         // waves per workgroup (4 or 8); a block is a tile of keys per wave
    int S;             // workgroups per (sequence, head) at most; 1 with several row groups: one takes them all in turn
    int rg_tiles;      // 16-row tiles of packed rows per workgroup (a row group)
    int n_rg;          // row groups per (sequence, head); 1 unless N is large
    uint64_t ranges;   // key ranges per row group at most, by the number of row groups that hold packed rows (attn_ranges)
    int usual;         // ... where the sequences of a batch differ in that number
    int sorted;        // long sequences first: more workgroups than the chip holds, of eight tiles per wave and more, and
                       // at most kOneStep sequences (us, ranked in steps of 64 / not at all: 8 x 5 tokens, H=4, 100 to 1500 keys,
                       // B=512 205 / 180; H=32, 100 to 1000 keys 1231 / 926)
    size_t counters_bytes;
    size_t total_bytes;
};

// Row groups of a head in the matrix-core kernel, as equal as whole 16-row tiles allow, and the tiles of each.
struct AttnGroups { int rg_tiles, n_rg; };
static inline AttnGroups attn_groups(int N)
{
    constexpr int kMaxTilesPerGroup = 3;    // as instantiated: a wave holds 32 accumulators per tile (D = 128)
    const int nq_all = (N + 15) / 16, n_rg = (nq_all + kMaxTilesPerGroup - 1) / kMaxTilesPerGroup;
    const int nq = (nq_all + n_rg - 1) / n_rg;
    return {nq, (nq_all + nq - 1) / nq};
}

// Key ranges per row group where n_act groups (1 to 8) hold packed rows: a byte each, 1 to 64.
__host__ __device__ inline int attn_ranges(uint64_t ranges, int n_act) { return (int)(ranges >> (8 * (n_act - 1))) & 0xff; }

// Bytes of the completion counters, in front of the partial results.  One workspace may serve calls planned for
// different contexts (ctx_bound of rd_tree_attn_bounded): a counter must never lie where another of these plans keeps
// partial results, so their room depends on the shape alone.
static inline size_t attn_counters_bytes(long long BH, int N)
{
    return ((size_t)BH * attn_groups(N).n_rg * sizeof(unsigned long long) + 255) / 256 * 256;
}

// Looks for the workgroups per head S with the shortest estimate of the launch, from n_rg (one per row group) up: S / n_act
// ranges of at most `per` of a head's nblk blocks, n_part of them with keys.  Those that leave the longest range at `per`
// blocks take no less time than the fewest of them, so only these are looked at (`every`: all; they agree).  est(S, per,
// n_part) gives microseconds; returns the best, and its S in *best_S, if it is below best_T, else best_T.
template <typename Est>
static inline double attn_search(int n_rg, int n_act, int nblk, bool every, double best_T, int *best_S, Est est)
{
    static const int forced_env = env_int("RD_ATTN_SPLITS", 0);
    const int most = (nblk < 64 ? nblk : 64) * n_rg;
    const int forced = forced_env > 0 && forced_env < n_rg ? n_rg : (forced_env < most ? forced_env : most);
    for (int S = n_rg, next; S <= most; S = next) {
        const int ranges = S / n_act, per = (nblk + ranges - 1) / ranges, n_part = (nblk + per - 1) / per;
        next = S + 1;
        if (forced <= 0 && !every) {
            if (per <= 1) next = most + 1;
            else if ((nblk + per - 2) / (per - 1) * n_act > S) next = (nblk + per - 2) / (per - 1) * n_act;
        }
        const double T = est(S, per, n_part);
        if (forced > 0 ? S == forced : T < best_T * (1 - 1e-9)) {
            best_T = T;
            *best_S = S;
        }
    }
    return best_T;
}

// Plan of the matrix-core kernel (rd_tree_attn_mfma.h), for contexts of up to Cmax keys: waves per workgroup and key ranges
// per row group, from an estimate of the launch time.  Lengths are upper bounds and the packed rows are not known at all
// here (distinct prefixes are taken to be 0.6 of the candidates' tokens, less of wide beams); the kernel starts no more row
// groups than hold packed rows and deals the tiles it finds to the ranges that the plan has for so many groups.  The constants
// are fitted to 1320 launches on MI355X (100 shapes, four and eight waves, 1 to 20 ranges), us, with r = row tiles that hold
// packed rows:
//   * a workgroup takes 2.8 (four waves) or 3.8 (eight), and 1.15 or 0.6 for at most one tile per wave, else 0.62 + 0.22 r or
//     0.85 + 0.25 r per tile of a wave (D = 64: 0.65 of that) and 0.7 r or 0.95 r where the waves' states meet;
//   * one eight-wave workgroup fills a compute unit, two of four waves do; more start as those retire;
//   * the workgroups that run at one time share 6.6 (four waves) or 5.9 TB/s of HBM, of which row groups of a range take one
//     share together, a compute unit gets 51 GB/s at most, and one with two workgroups takes twice as long as one with one (the
//     rest of the chip then idles, which leaves the others more: half of that is counted); latency and bandwidth overlap but
//     for where they are close (fourth root of the sum of fourth powers);
//   * more than one range adds a merge: 1.6, the partial results read by one compute unit at 48 GB/s, and all of them
//     written and read at 4.6 TB/s.
// Several row groups take four waves: their number is only guessed here, and where one more than that no longer fits the chip
// eight waves take two rounds (H=32, C=1777, 350 tokens: 21.9 us with 4 groups of packed rows, 36.6 with 5; four waves 21.5
// and 29.7).  Eight where all of them fit the chip and a head has a tile for each wave at most, but more than four of them
// (B=3, H=8, C=154, 88 tokens: 9.2 us by four waves, 7.4 by eight; B=2, H=4, C=70, 84 tokens 8.8 and 6.5; but D=64, B=1, H=8,
// C=66, 72 tokens 4.65 and 4.8).  Over 100 shapes the choice is 1.4 % slower than the best of the 18 in the mean, 17 % at worst.
static inline AttnPlan attn_plan_make(int B, int H, int N, int D, int Cmax, bool every = false)
{
    const long long BH = (long long)B * H;
    const size_t counters_bytes = attn_counters_bytes(BH, N);
    const int nq = attn_groups(N).rg_tiles, n_rg = attn_groups(N).n_rg;
    const double guess = 0.6 * N < 20 + 0.42 * N ? 0.6 * N : 20 + 0.42 * N, scale = D == 128 ? 1.0 : 0.65;
    const int n_guess = (int)ceil(guess / (16 * nq));
    static const int waves_env = env_int("RD_ATTN_WAVES", 0), forced_env = env_int("RD_ATTN_SPLITS", 0);
    struct Choice {
        double T;
        int R, sorted;
    };
    // The best number of ranges where n_act row groups hold `rows` packed rows; `usual` instead (if there is one) unless the
    // estimate is less than `margin` of that one's.
    auto choose = [&](int waves, int n_act, double rows, int usual, double margin) {
        const double r = n_act > 1 ? nq : ceil(rows / 16), part = r * 16 * (2 + D) * sizeof(float);
        const int tiles = (Cmax + 31) / 32 + ((int)rows + 31) / 32;
        const int nblk = tiles > waves ? (tiles + waves - 1) / waves : 1, most = nblk < 64 ? nblk : 64;
        const int forced = forced_env > most ? most : forced_env;
        const double t_tile = scale * (waves == 8 ? 0.85 + 0.25 * r : 0.62 + 0.22 * r), t_meet = scale * r * (waves == 8 ? 0.95 : 0.7);
        const double t_wg = waves == 8 ? 3.8 : 2.8, t_one = waves == 8 ? 0.6 : 1.15, rate = waves == 8 ? 5.9e6 : 6.6e6;
        const long long slots = waves == 8 ? 256 : 512;
        Choice best = {1e30, 1, 0};
        double T_usual = 1e30;
        for (int R = 1; R <= most; ++R) {
            const int per = (tiles + R - 1) / R, steps = (per + waves - 1) / waves;
            // more ranges with as many tiles per wave take no less time: only the fewest of them are looked at (`every`: all; they agree)
            if (!every && forced <= 0 && R > 1 && R != usual && steps == ((tiles + R - 2) / (R - 1) + waves - 1) / waves) continue;
            const double t_lat = t_wg + (steps == 1 ? t_one : steps * t_tile + t_meet);
            const double all = (double)(steps * waves < tiles ? steps * waves : tiles) * 32 * D * 4;      // of K and V, for a workgroup
            const long long wgs = (BH + 7) / 8 * 8 * n_act * R, full = wgs / slots, rest = wgs % slots;
            auto round = [&](long long n) {
                const long long per_cu = (n + 255) / 256;
                const double sharing = ((n < 256 ? n : 256) + (double)n / per_cu) / 2;
                const double t_hbm = per_cu * all / n_act * sharing / rate, t_cu = per_cu * all / 51e3, t_bw = t_hbm > t_cu ? t_hbm : t_cu;
                const double l2 = t_lat * t_lat, b2 = t_bw * t_bw;
                return sqrt(sqrt(l2 * l2 + b2 * b2));
            };
            double T = full * round(slots) + (rest ? round(rest) : 0.0);
            if (R > 1) T += 1.6 + R * part / 48e3 + 2.0 * (double)BH * n_act * R * part / 4.6e6;
            if (forced > 0 ? R == forced : T < best.T * (1 - 1e-9)) best = {T, R, B > 1 && B <= kOneStep && wgs > slots && steps >= 8};
            if (R == usual) T_usual = T;
        }
        if (T_usual * margin <= best.T) best.R = usual;
        return best;
    };
    const int ctx_tiles = (Cmax + 31) / 32;
    const bool eight = n_rg == 1 || ((BH + 7) / 8 * 8 * n_rg <= 256 && ctx_tiles >= (D == 128 ? 3 : 4) && ctx_tiles + (N + 31) / 32 <= 8);
    AttnPlan plan = {};
    Choice best = {1e30, 1, 0};
    for (int waves = 8; waves >= 4; waves -= 4) {
        if (waves_env ? waves != waves_env : waves == 8 && !eight) continue;
        const Choice c = choose(waves, n_guess, guess, 0, 1.0);
        if (c.T < best.T * (1 - 1e-9)) {
            best = c;
            plan.waves = waves;
        }
    }
    // The kernel finds how many row groups hold packed rows and takes the ranges of that number: those of the guess unless the
    // estimate promises 7 % (it is not exact to less: 30 x 5 tokens, H=32, C=2048, 120 packed rows 23.2 us with the guess's four,
    // 24.0 with five, where it promises 4 %).  us with the guess's ranges for all -> these, H=32: 70 x 5 tokens, C=1777, 30
    // packed rows 18.6 -> 15.0, 96 20.8 -> 17.4, 200 29.9 -> 25.8; C=4096, 200 47.6 -> 39.2.
    // Sequences that differ in the number of their groups take the guess's (`usual`), and so do more than kOneStep of them: ranges that
    // suit a launch whose heads are all alike put workgroups of one sequence on the compute units that the walks of another hold
    // (us with the guess's / each sequence's own: B=4, H=40, 16 x 5, C=4096, 27 to 60 packed rows 65.8 / 88.5; B=2, H=32, 70 x 5,
    // C=3000, 40 and 300 42.5 / 55.9; B=8, H=8, 70 x 5, C=4000, 20 to 300 50.4 / 83.1).  Where all have as many groups the gain is as
    // for one (B=2, H=32, 50 x 5, C=3000, 40 packed rows each 41.1 -> 29.4, contexts of 1000 to 3000 36.8 -> 26.0; B=4, H=40, 30 x 5, C=4000,
    // 130 each 114 -> 92.5), but for more ranges in a launch that does not fit the chip at once, which pay only where the
    // contexts are alike too (B=4, H=40, 16 x 5, 60 each, C=4096 94.8 -> 84.0, C=1000 to 4096 56.1 -> 60.0): not taken.
    int most = 1;
    for (int n = 1; n <= n_rg; ++n) {
        int R = n == n_guess || B > kOneStep ? best.R : choose(plan.waves, n, (n - 0.5) * 16 * nq, best.R, 0.93).R;
        if (B > 1 && R > best.R && (BH + 7) / 8 * 8 * n * R > (plan.waves == 8 ? 256 : 512)) R = best.R;
        plan.ranges |= (uint64_t)R << (8 * (n - 1));
        const int either = R > best.R ? R : best.R;
        plan.S = either * n > plan.S ? either * n : plan.S;
        most = either > most ? either : most;
    }
    plan.usual = best.R;
    plan.sorted = best.sorted;
    // Hundreds of sequences: finding a workgroup's place in the batch (0.5 us per 256 sequences and workgroup, also of those
    // that then have nothing to do) costs more than reading K and V once per row group where contexts are short beside the batch.
    // us, by places / one workgroup per head, which takes the row groups in turn (one group of packed rows; two): 16 x 5 tokens,
    // H=4, up to 300 keys, B=1024 130 / 110 and 169 / 158, B=2048 307 / 211 and 379 / 310; H=8, B=600, up to 1000 keys 366 / 356
    // and 404 / 456.
    // (A launch holds fewer than 2^32 threads.)
    const bool many = B > 256 && BH >= 2048 && (long long)n_rg * Cmax <= B, too_many = BH * n_rg >= 1ll << 24;
    if (n_rg > 1 && most == 1 && ((many && !plan.sorted) || too_many)) plan.S = 1;
    plan.rg_tiles = nq;
    plan.n_rg = n_rg;
    plan.counters_bytes = counters_bytes;
    plan.total_bytes = counters_bytes + (most > 1 ? ((size_t)BH * plan.S * (size_t)(nq * 16 * (2 + D)) * sizeof(float) + 255) / 256 * 256 : 0);
    return plan;
}

// Microseconds that merging n_part partial results of `part` bytes each takes: written and read back, the reading by one
// compute unit at 50 GB/s.
static inline double attn_merge_us(long long units, int n_part, double part)
{
    return n_part > 1 ? 1.5 + n_part * part / 50e3 + 2.0 * (double)units * n_part * part / 4e6 : 0.0;
}

// Plan of the fp32 kernel (rd_tree_attn_f32.hip; row groups of one tile): workgroups per head, estimated as above.  A
// workgroup is eight waves of 16-key tiles; a block of 128 keys takes 3.0 us (D = 128) or half of that, a compute
// unit reads 40 GB/s, the chip 5 TB/s.
static inline AttnPlan attn_plan_make_f32(int B, int H, int N, int D, int Cmax, bool every = false)
{
    AttnPlan best = {};
    const long long BH = (long long)B * H;
    const double rows = 0.6 * N, t_blk = D == 128 ? 3.0 : 1.5, part = 16.0 * (2 + D) * sizeof(float);
    const int tiles = (Cmax + 15) / 16 + ((int)rows + 15) / 16, nblk = tiles > 8 ? (tiles + 7) / 8 : 1;
    const int n_rg = (N + 15) / 16, n_act = rows > 16 ? (int)((rows + 15) / 16) : 1;
    best.waves = 8;
    best.rg_tiles = 1;
    best.n_rg = n_rg;
    best.ranges = 1;       // (not used: workgroups are dealt by S)
    attn_search(n_rg, n_act, nblk, every, 1e30, &best.S, [&](int wgs_per_head, int per, int n_part) {
        const double t_lat = 1.5 + per * t_blk, bytes = (double)(per * 8 < tiles ? per * 8 : tiles) * 16 * D * 8;
        const long long wgs = (BH + 7) / 8 * 8 * wgs_per_head, full = wgs / 256, rest = wgs % 256;
        auto round = [&](long long n) {
            const double t_bw = bytes / (5e6 / n < 40e3 ? 5e6 / n : 40e3);
            return sqrt(t_lat * t_lat + t_bw * t_bw);
        };
        return full * round(256) + (rest ? round(rest) : 0.0) + attn_merge_us(BH * n_act, n_part, part);
    });
    best.counters_bytes = ((size_t)BH * n_rg * sizeof(unsigned long long) + 255) / 256 * 256;
    best.total_bytes = best.counters_bytes + ((size_t)BH * (best.S > 2 ? best.S : 2) * (size_t)(16 * (2 + D)) * sizeof(float) + 255) / 256 * 256;
    return best;
}

// A search takes 0.4 us, up to 2 at few heads and long contexts (4 with every number of workgroups looked at); a program
// calls with few shapes at a time (the models it serves, their batches, a context bound that grows), so each thread keeps
// its last eight plans, the oldest of which makes room.
static inline AttnPlan attn_plan(int B, int H, int N, int D, int Cmax, bool f32 = false)
{
    constexpr int kKept = 8;
    struct Entry {
        int B, H, N, D, Cmax, f32;      // B = 0: empty
        AttnPlan plan;
    };
    static thread_local Entry kept[kKept] = {};
    static thread_local int oldest = 0;
    for (const Entry &e : kept)
        if (e.B == B && e.H == H && e.N == N && e.D == D && e.Cmax == Cmax && e.f32 == (int)f32) return e.plan;
    Entry &e = kept[oldest];
    oldest = (oldest + 1) % kKept;
    e = {B, H, N, D, Cmax, (int)f32, f32 ? attn_plan_make_f32(B, H, N, D, Cmax) : attn_plan_make(B, H, N, D, Cmax)};
    return e.plan;
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
    int B, H, N, Cmax, S, words;
    int n_rg;      // row groups per (sequence, head) (each is NQ*16 rows of the kernel's template)
    // (`usual` fills a gap of the layout: behind `ranges` the arguments took one load more, and a launch with rotation 0.25 us)
    int usual;     // key ranges per row group at most where sequences differ in the number of groups with packed rows
    uint64_t ranges;   // ... by that number where they do not (attn_ranges)
    int sorted;    // workgroups of long sequences first
    float scale_log2e;
    // rotary embedding fused into the call (rd_tree_attn_rope); unused (null) otherwise
    const int32_t *position_ids;   // [B, N]
    const float *cos_tab, *sin_tab;   // [max_pos, D/2]
    int max_pos;
    void *k_rot;                   // [B,H,N,D] rotated packed keys (output), or null
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

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

// max / sum over the four lanes l, l^16, l^32, l^48 (the four key groups of a score tile's column) with the gfx950
// lane-swap instructions: each gives a lane the pair {x[l], x[l^k]}.
__device__ __forceinline__ float quad_max(float x)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_sum(float x)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

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

}  // namespace rd
