// Device-side helpers shared by the RADAR kernels (gfx950, 64-wide wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/radar.h"

namespace radar {

constexpr int kWave = 64;

// ---------------------------------------------------------------- ordering
// Monotone map float -> uint32 (larger float <=> larger integer); -0.0 is folded
// onto +0.0 first so that it ties with it, as a float comparison would.
__device__ __forceinline__ uint32_t ord_of(float x) {
    x = x + 0.0f;
    uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float float_of_ord(uint32_t o) {
    uint32_t b = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
    return __uint_as_float(b);
}
// One 64-bit key per (value, index): comparing keys as unsigned integers gives
// "value descending, index ascending" when the larger key wins.
__device__ __forceinline__ uint64_t make_key(float x, uint32_t idx) {
    return (uint64_t(ord_of(x)) << 32) | uint64_t(~idx);
}
__device__ __forceinline__ uint32_t key_index(uint64_t key) { return ~uint32_t(key); }
__device__ __forceinline__ float key_value(uint64_t key) { return float_of_ord(uint32_t(key >> 32)); }

// ------------------------------------------------------------ DPP reductions
// dpp_ctrl: quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E, row_half_mirror = 0x141,
// row_mirror = 0x140.  After the four steps every lane of a 16-lane row holds
// the row's reduction; the four rows are then combined through scalar reads.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    uint32_t lo = dpp_u32<CTRL>(uint32_t(v));
    uint32_t hi = dpp_u32<CTRL>(uint32_t(v >> 32));
    return (uint64_t(hi) << 32) | lo;
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __uint_as_float(dpp_u32<CTRL>(__float_as_uint(v)));
}

// ------------------------------------------------------------------- rows of any alignment
// Rows of V floats with V % 4 != 0 start at any multiple of 4 bytes, which is all that a 16-byte load of global memory needs
// on this chip: a wavefront's request covers one cache line more.  Four of a row of n >= 4 from i on; what would
// reach past the row's end is read from n - 4 on, and place_row_end() brings it to its place.
__device__ __forceinline__ float4 load4_of_row(const float *row, int i, int n) {
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    const f32x4_any v = *reinterpret_cast<const f32x4_any *>(reinterpret_cast<const char *>(row) + (uint32_t)min(i, n - 4) * 4u);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 load4_of_short_row(const float *row, int n) {   // of one shorter than four, from its start
    return make_float4(row[0], row[min(1, n - 1)], row[min(2, n - 1)], row[n - 1]);
}
// x(g, 0 ... 3): four from first + g * step on, a multiple of 4, as load4_of_row left them.  Entries from n on are the caller's to mask.
template <int G, typename X>
__device__ __forceinline__ void place_row_end(X &&x, int first, int step, int n) {
    const int by = n >= 4 ? -n & 3 : 0;                            // how far the last four were moved
    auto at_end = [&](int g) { return (unsigned int)(n - 1 - (first + g * step)) < 3u; };
    if (by == 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const bool c = at_end(g);
            x(g, 0) = c ? x(g, 1) : x(g, 0); x(g, 1) = c ? x(g, 2) : x(g, 1); x(g, 2) = c ? x(g, 3) : x(g, 2);
        }
    } else if (by == 2) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const bool c = at_end(g);
            x(g, 0) = c ? x(g, 2) : x(g, 0); x(g, 1) = c ? x(g, 3) : x(g, 1);
        }
    } else if (by == 3) {
#pragma unroll
        for (int g = 0; g < G; ++g) x(g, 0) = at_end(g) ? x(g, 3) : x(g, 0);
    }
}

__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
    return (uint64_t(readlane_u32(uint32_t(v >> 32), lane)) << 32) | readlane_u32(uint32_t(v), lane);
}
__device__ __forceinline__ float readlane_f32(float v, int lane) {
    return __uint_as_float(readlane_u32(__float_as_uint(v), lane));
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, dpp_u32<0xB1>(v));
    v = max(v, dpp_u32<0x4E>(v));
    v = max(v, dpp_u32<0x141>(v));
    v = max(v, dpp_u32<0x140>(v));
    uint32_t a = max(readlane_u32(v, 0), readlane_u32(v, 16));
    uint32_t b = max(readlane_u32(v, 32), readlane_u32(v, 48));
    return max(a, b);
}
__device__ __forceinline__ uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    v = max_u64(v, dpp_u64<0xB1>(v));
    v = max_u64(v, dpp_u64<0x4E>(v));
    v = max_u64(v, dpp_u64<0x141>(v));
    v = max_u64(v, dpp_u64<0x140>(v));
    uint64_t a = max_u64(readlane_u64(v, 0), readlane_u64(v, 16));
    uint64_t b = max_u64(readlane_u64(v, 32), readlane_u64(v, 48));
    return max_u64(a, b);
}
__device__ __forceinline__ float wave_max_f32(float v) {
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    v = fmaxf(v, dpp_f32<0x141>(v));
    v = fmaxf(v, dpp_f32<0x140>(v));
    float a = fmaxf(readlane_f32(v, 0), readlane_f32(v, 16));
    float b = fmaxf(readlane_f32(v, 32), readlane_f32(v, 48));
    return fmaxf(a, b);
}
// Sum with a fixed association order (bit-reproducible from run to run).
__device__ __forceinline__ float wave_sum_f32(float v) {
    v = v + dpp_f32<0xB1>(v);
    v = v + dpp_f32<0x4E>(v);
    v = v + dpp_f32<0x141>(v);
    v = v + dpp_f32<0x140>(v);
    float a = readlane_f32(v, 0) + readlane_f32(v, 16);
    float b = readlane_f32(v, 32) + readlane_f32(v, 48);
    return a + b;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
    auto step = [](double x, uint64_t moved) { return x + __longlong_as_double((long long)moved); };
    v = step(v, dpp_u64<0xB1>((uint64_t)__double_as_longlong(v)));
    v = step(v, dpp_u64<0x4E>((uint64_t)__double_as_longlong(v)));
    v = step(v, dpp_u64<0x141>((uint64_t)__double_as_longlong(v)));
    v = step(v, dpp_u64<0x140>((uint64_t)__double_as_longlong(v)));
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const double a0 = __longlong_as_double((long long)readlane_u64(b, 0));
    const double a1 = __longlong_as_double((long long)readlane_u64(b, 16));
    const double a2 = __longlong_as_double((long long)readlane_u64(b, 32));
    const double a3 = __longlong_as_double((long long)readlane_u64(b, 48));
    return (a0 + a1) + (a2 + a3);
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    return __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(v), lane));
}

// Inclusive prefix sum over the lanes of a wavefront by DPP moves (shift by 1, 2, 4, 8 inside each
// 16-lane row, then the row totals are carried into the following rows); fixed association order.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_take_f64(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    // lanes without a source lane, and rows outside ROW_MASK, receive 0
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_scan_f64(double v) {
    v += dpp_take_f64<0x111, 0xF>(v);             // row_shr:1
    v += dpp_take_f64<0x112, 0xF>(v);             // row_shr:2
    v += dpp_take_f64<0x114, 0xF>(v);             // row_shr:4
    v += dpp_take_f64<0x118, 0xF>(v);             // row_shr:8
    v += dpp_take_f64<0x142, 0xA>(v);             // row_bcast:15 -> rows 1 and 3
    v += dpp_take_f64<0x143, 0xC>(v);             // row_bcast:31 -> rows 2 and 3
    return v;
}
// The same for 32-bit whole numbers.
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);
    return v;
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }
__device__ __forceinline__ int wave_id() { return (int)(threadIdx.x >> 6); }

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Orders LDS traffic between the lanes of one wavefront (a lane reads what another
// lane of the same wavefront wrote earlier in program order).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------- cross-workgroup hand-over
// Results that one workgroup leaves for another workgroup of the SAME launch
// (partials merged by the last arriver) travel through device-scope accesses:
// every such store and load carries agent scope, so it is written through /
// fetched past the per-XCD L2 on its own.  This replaces agent-scope fences,
// which on this part write back and invalidate a whole L2 (measured: ~8 us per
// fence against ~0.1 us for the scoped accesses).  Protocol:
//   producer: store_shared_result(...) for everything it hands over;
//             publish_then_ticket() = wait until this lane's stores are
//             acknowledged (vmcnt 0), workgroup barrier, one relaxed device-
//             scope fetch-add by lane 0;
//   consumer (the workgroup whose ticket is the last): load_shared_result(...)
//             only -- it never reads handed-over data through a plain load.
template <typename T>
__device__ __forceinline__ T load_shared_result(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void store_shared_result(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Returns, to every lane of the workgroup, the value the counter had before this
// workgroup's arrival.  `flag` is one int of LDS.  All lanes must call it.
__device__ __forceinline__ unsigned int publish_then_ticket(unsigned int *counter, unsigned int *flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        *flag = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return *flag;
}

// ------------------------------------------------- arguments that are needed later
// A kernel's leading scalar arguments are in registers when it starts; the rest is a block behind them (type Args, the last parameter), every
// cache line of which is a round trip of 0.3 us.  Left to itself the compiler loads all of it at the start and waits for it,
// to work out or to move away what is needed at the end, before the first loads from memory are asked for.  This gives the block's
// address to loads that come after it in the program.  Lead: the leading parameters and the block, in order.
template <typename Args>
using ArgBlock = const __attribute__((address_space(4))) Args *;
template <typename Args>
__device__ __forceinline__ ArgBlock<Args> args_from_here(size_t at) {
    auto p = (ArgBlock<Args>)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + at);
    asm volatile("" : "+s"(p) :: "memory");
    return p;
}

// A word that is the same for the whole workgroup and that nothing writes while the kernel runs: by a scalar load wherever it stands (behind
// args_from_here the compiler would take a vector load, and branches on the word for divergent ones).
__device__ __forceinline__ int32_t uniform_word(const int32_t *p, int i) { return ((const __attribute__((address_space(4))) int32_t *)p)[i]; }

}  // namespace radar
