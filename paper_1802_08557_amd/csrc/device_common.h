// device_common.h -- small device helpers shared by the simplex kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "internal.h"

namespace lpb {

constexpr int kLE = 0, kGE = 1, kEQ = 2;
constexpr int kOptimal = 0, kInfeasible = 1, kUnbounded = 2, kIterLimit = 3, kNumerical = 4,
              kInvalid = 5;
constexpr int kBig = 0x7fffffff;
constexpr int kRowNeg = 1, kRowDead = 8, kRowPad = 16;
// Certificate outcome bits (stats[5]); the values of LP_CERT_* in lpbatch.h.
constexpr int LP_CERT_PRIMAL_OK_BIT = 1, LP_CERT_DUAL_OK_BIT = 2, LP_CERT_RAY_OK_BIT = 4,
              LP_CERT_SINGULAR_BIT = 8, LP_CERT_INFEASIBLE_OK_BIT = 16;

// f(std::integral_constant<int, B>) ... f(std::integral_constant<int, E - 1>):
// a loop over register arrays whose indices are constants from the start.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>());
        static_for<B + 1, E>(f);
    }
}

template <typename T> __device__ __forceinline__ T t_inf();
template <> __device__ __forceinline__ float t_inf<float>() { return __builtin_inff(); }
template <> __device__ __forceinline__ double t_inf<double>() { return __builtin_inf(); }

// Lanes where v holds.  (__ballot takes an integer: the condition is first
// turned into one and compared again, two more instructions.)
__device__ __forceinline__ uint64_t ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }

// Wavefront-uniform read of lane l's value (l must be wavefront-uniform).
__device__ __forceinline__ int lane_get(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_get(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_get(double v, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// A register copy the compiler cannot fold back into its source, so the
// source's register is free for a new load once the copy is made (a value
// prefetched for the next work item can then land where the current one was).
__device__ __forceinline__ double fresh_copy(double v)
{
    double r;
    asm("v_mov_b64 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(v >> 32)));
    return int64_t((uint64_t(hi) << 32) | lo);
}
template <typename P>
__device__ __forceinline__ P *uniform_ptr(P *p)
{
    return reinterpret_cast<P *>(uniform64(reinterpret_cast<int64_t>(p)));
}

// Buffer descriptor over `bytes` bytes from p (p wavefront-uniform): the
// hardware range check makes loads at offsets >= bytes return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_over(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(const_cast<void *>(p)), short(0), bytes, 0x00020000);
}
__device__ __forceinline__ double buffer_f64(__amdgpu_buffer_rsrc_t rs, int byte_off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, byte_off, 0, 0));
}

// ---- DPP / permlane reductions (all 64 lanes must be active) ---------------
// Lane patterns (checked on gfx950): quad_perm [1,0,3,2] and [2,3,0,1] swap
// neighbours at distance 1 and 2, row_half_mirror reverses each group of 8,
// row_mirror each row of 16; permlane16_swap(v, v) yields {even-row value,
// odd-row value} and permlane32_swap(v, v) {low-half value, high-half value}
// at the lane's own position.  After the six steps every lane holds the result.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}

struct Pair32 { int a, b; };

__device__ __forceinline__ Pair32 swap16(int v)
{
    auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return {int(p[0]), int(p[1])};
}
__device__ __forceinline__ Pair32 swap32(int v)
{
    auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return {int(p[0]), int(p[1])};
}

__device__ __forceinline__ int wave_min_i(int v)
{
    v = min(v, dpp_i<0xB1>(v));
    v = min(v, dpp_i<0x4E>(v));
    v = min(v, dpp_i<0x141>(v));
    v = min(v, dpp_i<0x140>(v));
    Pair32 p = swap16(v);
    v = min(p.a, p.b);
    p = swap32(v);
    return min(p.a, p.b);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f(double v)
{
    return __hiloint2double(dpp_i<CTRL>(__double2hiint(v)), dpp_i<CTRL>(__double2loint(v)));
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}

__device__ __forceinline__ void swap16_f(double v, double &a, double &b)
{
    Pair32 lo = swap16(__double2loint(v)), hi = swap16(__double2hiint(v));
    a = __hiloint2double(hi.a, lo.a);
    b = __hiloint2double(hi.b, lo.b);
}
__device__ __forceinline__ void swap32_f(double v, double &a, double &b)
{
    Pair32 lo = swap32(__double2loint(v)), hi = swap32(__double2hiint(v));
    a = __hiloint2double(hi.a, lo.a);
    b = __hiloint2double(hi.b, lo.b);
}
__device__ __forceinline__ void swap16_f(float v, float &a, float &b)
{
    Pair32 p = swap16(__float_as_int(v));
    a = __int_as_float(p.a);
    b = __int_as_float(p.b);
}
__device__ __forceinline__ void swap32_f(float v, float &a, float &b)
{
    Pair32 p = swap32(__float_as_int(v));
    a = __int_as_float(p.a);
    b = __int_as_float(p.b);
}

// Exact minimum / maximum of a floating-point value over the wavefront (no NaN).
template <typename T>
__device__ __forceinline__ T wave_min_f(T v)
{
    v = fmin(v, dpp_f<0xB1>(v));
    v = fmin(v, dpp_f<0x4E>(v));
    v = fmin(v, dpp_f<0x141>(v));
    v = fmin(v, dpp_f<0x140>(v));
    T a, b;
    swap16_f(v, a, b);
    v = fmin(a, b);
    swap32_f(v, a, b);
    return fmin(a, b);
}
template <typename T>
__device__ __forceinline__ T wave_max_f(T v)
{
    v = fmax(v, dpp_f<0xB1>(v));
    v = fmax(v, dpp_f<0x4E>(v));
    v = fmax(v, dpp_f<0x141>(v));
    v = fmax(v, dpp_f<0x140>(v));
    T a, b;
    swap16_f(v, a, b);
    v = fmax(a, b);
    swap32_f(v, a, b);
    return fmax(a, b);
}

// Unsigned minimum / maximum over the wavefront (all 64 lanes active).
__device__ __forceinline__ uint32_t wave_min_u(uint32_t v)
{
    v = min(v, uint32_t(dpp_i<0xB1>(int(v))));
    v = min(v, uint32_t(dpp_i<0x4E>(int(v))));
    v = min(v, uint32_t(dpp_i<0x141>(int(v))));
    v = min(v, uint32_t(dpp_i<0x140>(int(v))));
    Pair32 p = swap16(int(v));
    v = min(uint32_t(p.a), uint32_t(p.b));
    p = swap32(int(v));
    return min(uint32_t(p.a), uint32_t(p.b));
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) { return ~wave_min_u(~v); }

// Lanes among `on` that hold the least (largest) value, as a mask; every value
// of an `on` lane is >= +0 and not NaN, so its bits order like an unsigned
// integer's.  FP64 compares high words first and low words only where those
// tie: one 32-bit reduction instead of a 64-bit one, whose every step is three
// dependent instructions.
__device__ __forceinline__ uint64_t wave_min_nonneg(bool on, float v)
{
    const uint32_t u = __float_as_uint(v);
    const uint32_t best = wave_min_u(on ? u : 0xffffffffu);
    return ballot(on && u == best);
}
__device__ __forceinline__ uint64_t wave_min_nonneg(bool on, double v)
{
    const uint32_t hi = uint32_t(__double2hiint(v)), lo = uint32_t(__double2loint(v));
    const uint32_t best = wave_min_u(on ? hi : 0xffffffffu);
    const uint64_t tied = ballot(on && hi == best);
    if (__builtin_expect(__popcll(tied) <= 1, 1)) return tied;
    const bool in = on && hi == best;
    const uint32_t low = wave_min_u(in ? lo : 0xffffffffu);
    return ballot(in && lo == low);
}
__device__ __forceinline__ uint64_t wave_max_nonneg(bool on, float v)
{
    const uint32_t u = __float_as_uint(v);
    const uint32_t best = wave_max_u(on ? u : 0u);
    return ballot(on && u == best);
}
__device__ __forceinline__ uint64_t wave_max_nonneg(bool on, double v)
{
    const uint32_t hi = uint32_t(__double2hiint(v)), lo = uint32_t(__double2loint(v));
    const uint32_t best = wave_max_u(on ? hi : 0u);
    const uint64_t tied = ballot(on && hi == best);
    if (__builtin_expect(__popcll(tied) <= 1, 1)) return tied;
    const bool in = on && hi == best;
    const uint32_t low = wave_max_u(in ? lo : 0u);
    return ballot(in && lo == low);
}

// The 16 x 16 x 4 matrix product of each tableau type.  Lane (q = lane / 16,
// lane % 16) holds column lane % 16 of the tile and, in component v, row
// mfma_row(q, v).
template <typename T> struct Tile;
template <> struct Tile<double> {
    using V = double __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mma(double a, double b, V c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};
template <> struct Tile<float> {
    using V = float __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mma(float a, float b, V c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <typename T>
__device__ __forceinline__ int mfma_row(int q, int v)
{
    return sizeof(T) == 8 ? q + 4 * v : 4 * q + v;
}

// Worker b of `workers` in a launch's work queue: its first two items are b and
// second(); later ones come from pop() (one lane) through item().
struct QueuePlace {
    int groups, g, members;
    __device__ __forceinline__ QueuePlace(int b, int workers)
    {
        groups = min(kQueues, workers);
        g = b % groups;
        members = (workers - g + groups - 1) / groups;
    }
    __device__ __forceinline__ int64_t second(int b) const { return b + int64_t(groups) * members; }
    // The counter is read here and used when the current LP is done.  (An
    // increment with wrap at 2^32 - 1 is a plain +1 here; unlike an add it is
    // not rewritten into a wavefront-combined atomic whose result is broadcast,
    // and waited for, right away.)
    __device__ __forceinline__ int pop(int32_t *queue) const
    {
        return int(atomicInc(reinterpret_cast<unsigned *>(queue + kQueueLine * g), 0xffffffffu));
    }
    __device__ __forceinline__ int64_t item(int popped) const
    {
        return g + int64_t(groups) * (2 * int64_t(members) + popped);
    }
};

// Waits until every memory access of this wavefront has returned, a queue
// counter popped ahead and not needed any more among them.
__device__ __forceinline__ void drain_memory() { __builtin_amdgcn_s_waitcnt(0); }

// Called once per workgroup (one thread, after drain_memory in every wavefront)
// when it leaves its work loop: the last workgroup to finish returns the
// launch's counters to 0 for the next launch on the stream.
__device__ __forceinline__ void finish_launch(int32_t *queue, int32_t *extra)
{
    if (!queue) return;
    const int groups = min(kQueues, int(gridDim.x)), g = int(blockIdx.x) % groups;
    const int members = (int(gridDim.x) - g + groups - 1) / groups;
    if (atomicAdd(queue + kQueueLine * g + 1, 1) != members - 1) return;
    if (atomicAdd(queue + kQueueLine * kQueues, 1) != groups - 1) return;
    for (int q = 0; q <= kQueues; ++q) {
        atomicExch(queue + kQueueLine * q, 0);
        atomicExch(queue + kQueueLine * q + 1, 0);
    }
    if (extra) atomicExch(extra, 0);
}

// A solve launch's arguments, read again from the kernel's argument segment where
// they are used: held in scalar registers from the start they spill.
typedef const __attribute__((address_space(4))) SolveArgs *LateArgs;
__device__ __forceinline__ LateArgs late_args()
{
    LateArgs p = (LateArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// Orders a wavefront's LDS and memory accesses around the call.  Lanes of one
// wavefront that exchange data through LDS need no instruction for it -- its accesses
// take effect in order -- but the compiler must not move one lane's read of another
// lane's entry across the store.
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint64_t lanemask_lt(int lane)
{
    return (uint64_t(1) << lane) - 1;
}

}  // namespace lpb
