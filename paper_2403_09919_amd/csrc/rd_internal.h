// Shared helpers of the rd library: argument and launch checks, tuning overrides, and the
// device-scope accesses with which workgroups hand partial results to one another.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <atomic>
#include "rd.h"

#define RD_WAVE 64

static inline bool rd_aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

static inline int rd_check_launch()
{
    return hipGetLastError() == hipSuccess ? RD_OK : RD_ERR_HIP;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every global
// load and store the wave has in flight, which turns each barrier after a global store into a
// round trip to memory.
__device__ __forceinline__ void rd_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Validates the (W, L) pair shared by rd_dedup and rd_accept.
static inline int rd_check_beam_shape(int B, int W, int L)
{
    if (B <= 0 || W <= 0 || L <= 0) return RD_ERR_INVALID_ARG;
    if (W > RD_MAX_W) return RD_ERR_UNSUPPORTED;
    if ((long long)W * (long long)L > RD_MAX_N) return RD_ERR_UNSUPPORTED;
    return RD_OK;
}

namespace rd {

// Integer environment override for tuning sweeps (unset or empty: the default).  Only builds made
// with -DRD_TUNING read the environment; in the product library every plan is fixed by its arguments.
static inline int env_int(const char *name, int dflt)
{
#ifdef RD_TUNING
    const char *v = getenv(name);
    return (v && *v) ? atoi(v) : dflt;
#else
    (void)name;
    return dflt;
#endif
}

// Raising a kernel's dynamic LDS limit is per kernel and per device; `done` (one per kernel) keeps
// a bit for each device already set up.  Returns RD_OK or RD_ERR_HIP.
static inline int ensure_dynamic_lds(const void *kernel, size_t bytes, std::atomic<unsigned long long> &done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return RD_ERR_HIP;
    const unsigned long long bit = 1ull << (dev & 63);
    if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return RD_OK;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return RD_ERR_HIP;
    if (dev < 64) done.fetch_or(bit, std::memory_order_release);
    return RD_OK;
}

// ---- exchange of partial results between workgroups -------------------------------------------
// Partial results (attention states, K-split sums of the drafter's layers) are written by one
// workgroup and read by another that may sit on a different XCD (each XCD has its own L2).  A
// device-wide release/acquire fence would write back and invalidate whole L2s on every
// workgroup, which costs far more than the kernel itself, so the
// exchange uses device-scope (write-through / cache-bypassing) relaxed atomic accesses for the
// data itself.  They are complete in one of two ways: the writer waits for its outstanding memory
// operations before it bumps the counter (wait_dev_stores: partial attention states, keys that several
// workgroups fold into), or the word itself says that it has been stored and the reader waits for it
// (poll: keys and totals that one workgroup stores).  Only these few KB per workgroup travel that way; the
// bulk streams use plain loads.
__device__ __forceinline__ void st_dev(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev2(float *p, float a, float b)
{
    unsigned long long u = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_dev(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_dev2(const float *p)
{
    const unsigned long long u =
        __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((unsigned)u), __uint_as_float((unsigned)(u >> 32)));
}

// 16 bytes, written through like the others: one store of whole lines, where two of 8 bytes each leave every second piece of
// a line to the other.  Nothing may rely on the 16 bytes arriving together.  A store that the compiler knows, not assembly:
// gfx950 needs two wait states between a store of more than 8 bytes and a vector write to its data registers, and up to eight
// in front of one whose data a matrix instruction wrote, and only the compiler sees what stands around it.
__device__ __forceinline__ void st_dev4(float *p, float a, float b, float c, float d)
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const u4 v = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
    __builtin_amdgcn_global_store_b128((u4 __attribute__((address_space(1))) *)p, v, "agent");
}
// Returns once every vector memory operation this wave has issued -- loads, stores and atomics without
// a return value alike, they share one counter -- has been acknowledged.  A device-scope store or atomic
// is acknowledged when it has been performed past the XCD's L2, where every other XCD can see it.  This
// is the release half of the exchange; a release FENCE at device scope would also write back the whole
// L2, which is what the exchange avoids.
__device__ __forceinline__ void wait_dev_stores() { asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); }

// Where nobody waits for a store before the counter is bumped, whoever sees the full count reads the word, which is 0 until the
// store arrives, until it is there.  The store has been issued by then and arrives within microseconds, so that the first read
// nearly always finds it.  The wait has an end all the same (some 50 ms): calls that overlap on one workspace may clear
// each other's words, and must end with wrong results, not hang.  Returns the last value read.
constexpr int kPolls = 1 << 16;
template <typename Read, typename There> __host__ __device__ __forceinline__ auto poll(Read read, There there)
{
    auto x = read();
    for (int i = 1; i < kPolls && !there(x); ++i) x = read();
    return x;
}

// ---- memory straight into LDS -------------------------------------------------------------------------
// Copies 1 KB of memory into LDS, 16 bytes per lane, without passing through registers: lane l's bytes come from
// base + off and land at lds + 16 l.  Complete when the wave's count of vector memory operations says so (wait_vm);
// loads return in the order they were issued.  The compiler knows nothing of these loads: whoever reads the bytes waits,
// and no wave ends or lets its LDS go with one under way.  (m0 holds the destination; nothing else here uses it.)
// Nor does it keep wait states in front of them: one between m0 and its use, and five where a vector instruction wrote the
// base's scalar registers (uniform, or a register that comes back from a vector register's lane).  A scalar copy of the base
// stands for both: the scalar unit waits for what it reads, and its own results may be used at once.  (Five empty slots
// instead: a step of eight layers, H=32, C=1777, 70 x 5 tokens 183.5 -> 185.5 us; so 193.2 -> 193.7 on another machine.)
__device__ __forceinline__ uintptr_t uniform(uintptr_t x)         // (in scalar registers, whatever it was computed in)
{
    return (uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) | (uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32;
}
__device__ __forceinline__ void dma16(uintptr_t base, uint32_t off, uint32_t lds)
{
    uintptr_t at;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0" : "=&s"(at) : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(off), "s"(uniform(base)) : "memory");
}
// The same from an address per lane.
__device__ __forceinline__ void dma16(uintptr_t lane_address, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(lane_address) : "memory");
}
// 4 bytes per lane, from base + off.
__device__ __forceinline__ void dma4(uintptr_t base, uint32_t off, uint32_t lds)
{
    uintptr_t at;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0" : "=&s"(at) : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(off), "s"(uniform(base)) : "memory");
}
// Returns when at most N of the wave's vector memory operations are outstanding.
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
// Returns when the wave's LDS reads but the last N are in registers (they return in order; scalar loads in flight only make the wait longer).
template <int N = 0> __device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory"); }

// ---- rows of any length in 16-byte loads --------------------------------------------------------------
// Rows of V floats start at multiples of 4 bytes only, unless V is a multiple of 4; global memory instructions of any
// width need no more.  (Scalar loads for such rows cost a vocabulary-wide pass two to three times its time.)
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
// Past a row's end addresses are pulled back.  No branches: an `if` on what was loaded becomes one here, which waits for
// every load in flight, load after load, in the workgroup that holds the row's end.
// Four entries from v on or, at the end of the row (n >= 4), its last four; *at: the first one's index.
__device__ __forceinline__ float4 row4_at(const float *row, int v, int n, int *at)
{
    const int a = *at = min(v, n - 4);
    const f4_any q = *reinterpret_cast<const f4_any *>(row + a);
    return make_float4(q[0], q[1], q[2], q[3]);
}
// The entries v .. v+3 that exist, -inf in place of the others; in any order.
__device__ __forceinline__ float4 row4_set(const float *row, int v, int n)
{
    int a;
    const float4 q = row4_at(row, v, n, &a);
    return make_float4(a < v ? -INFINITY : q.x, a + 1 < v ? -INFINITY : q.y, a + 2 < v ? -INFINITY : q.z, a + 3 < v ? -INFINITY : q.w);
}
// Entries v .. v+3, -inf past the end.
__device__ __forceinline__ float4 row4(const float *row, int v, int n)
{
    int a;
    const float4 q = row4_at(row, v, n, &a);
    const int d = v - a;
    const bool one = d & 1, two = d & 2, all = d > 3;
    const float x = one ? q.y : q.x, y = one ? q.z : q.y, z = one ? q.w : q.z, w = one ? -INFINITY : q.w;
    return make_float4(all ? -INFINITY : (two ? z : x), all ? -INFINITY : (two ? w : y), all || two ? -INFINITY : z, all || two ? -INFINITY : w);
}

// ---- reductions over the 64 lanes, the same value in every lane --------------------------------------
// Data-parallel primitives inside rows of 16 and the gfx950 lane swaps across them: about ten instructions, where
// __shfl_xor is six round trips through LDS.
template <int kCtrl> __device__ __forceinline__ float dpp(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)__float_as_uint(x), (int)__float_as_uint(x), kCtrl, 0xf, 0xf, false));
}
// K values at once, over aligned groups of `lanes` lanes, a power of two that is the same in the whole wave.
template <int K, typename Op> __device__ __forceinline__ void group_reduce(float (&x)[K], int lanes, Op op)
{
    auto each = [&](auto other) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = op(x[k], other(x[k]));
    };
    if (lanes > 1) each([](float a) __attribute__((always_inline)) { return dpp<0xB1>(a); });      // quad_perm [1,0,3,2]: lane ^ 1
    if (lanes > 2) each([](float a) __attribute__((always_inline)) { return dpp<0x4E>(a); });      // quad_perm [2,3,0,1]: lane ^ 2
    if (lanes > 4) each([](float a) __attribute__((always_inline)) { return dpp<0x141>(a); });     // row_half_mirror: the other quad of the 8
    if (lanes > 8) each([](float a) __attribute__((always_inline)) { return dpp<0x140>(a); });     // row_mirror: the other half of the 16
    if (lanes > 16) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[k]), __float_as_uint(x[k]), false, false);
            x[k] = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
        }
    }
    if (lanes > 32) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[k]), __float_as_uint(x[k]), false, false);
            x[k] = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
        }
    }
}
template <typename Op> __device__ __forceinline__ float wave_reduce(float x, Op op)
{
    float v[1] = {x};
    group_reduce(v, 64, op);
    return v[0];
}
__device__ __forceinline__ float wave_reduce_max(float x) { return wave_reduce(x, [](float a, float b) { return fmaxf(a, b); }); }
// (non-negative integers below 2^31: their order is that of their bits)
__device__ __forceinline__ uint32_t wave_reduce_min_u(uint32_t x)
{
    return __float_as_uint(wave_reduce(__uint_as_float(x), [](float a, float b) {
        return __uint_as_float(min(__float_as_uint(a), __float_as_uint(b)));
    }));
}
// (integers from 0 on)
__device__ __forceinline__ int wave_reduce_max_i(int x)
{
    return __float_as_int(wave_reduce(__int_as_float(x), [](float a, float b) __attribute__((always_inline)) {
        return __int_as_float(max(__float_as_int(a), __float_as_int(b)));
    }));
}
__device__ __forceinline__ float wave_reduce_sum(float x) { return wave_reduce(x, [](float a, float b) { return a + b; }); }

// Length of the run of ones in a bit set from bit `first` on, at most L: a candidate's accepted prefix, where the candidates'
// tokens are a bit each in row-major order.  In one word, and in several.
__device__ __forceinline__ int accepted_run(uint64_t bits, int first, int L)
{
    const uint64_t zeros = ~(bits >> first);
    return min(zeros ? __builtin_ctzll(zeros) : 64, L);
}
__device__ __forceinline__ int accepted_run(const unsigned long long *bits, int first, int L)
{
    int len = 0;
    for (int run = 64; run > 0 && len < L; len += run) {
        const int pos = first + len, left = min(64 - (pos & 63), L - len);
        run = accepted_run(bits[pos >> 6], pos & 63, left);
        if (run < left) return len + run;
    }
    return len;
}

}  // namespace rd

// Optional phase timestamps for tuning builds (-DRD_TRACE): thread 0 of every workgroup stores
// the constant-rate wall clock at a few points into a caller-supplied buffer (one per source file).
#ifdef RD_TRACE
#define RD_TRACE_DEFINE(setter)                                                                   \
    __device__ unsigned long long *rd_trace_buf = nullptr;                                        \
    extern "C" int setter(unsigned long long *p)                                                  \
    {                                                                                             \
        return hipMemcpyToSymbol(HIP_SYMBOL(rd_trace_buf), &p, sizeof(p)) == hipSuccess ? 0 : -4; \
    }
#define RD_TR(i)                                                                                                   \
    do {                                                                                                           \
        if (threadIdx.x == 0 && rd_trace_buf)                                                                      \
            rd_trace_buf[((size_t)blockIdx.x + (size_t)gridDim.x * (blockIdx.y + (size_t)gridDim.y * blockIdx.z)) * 16 + (i)] = wall_clock64(); \
    } while (0)
#else
#define RD_TRACE_DEFINE(setter)
#define RD_TR(i) do { } while (0)
#endif
