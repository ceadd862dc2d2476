// What the kernels share at the level of a wave: register vector types, loads that go straight to LDS, folds over the lanes.
#pragma once
#include <utility>

#include "common.h"

namespace hr {

// compile-time loop: f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N-1>)
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
// 16 bytes as a register vector (a struct such as HIP's uint4 is copied with memcpy semantics,
// which can pin a local array of them to scratch memory)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// The lane number made anew where it is used.  What is computed from lane_id() does not change inside a loop, so the
// compiler computes it before the loop and keeps it in registers for the whole of it; in paths that are taken once in
// many blocks a few instructions are cheaper than registers that the multiplication has not got.
__device__ __forceinline__ int lane_now()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// value of lane ^ 8 (the other half of a row of 16 lanes: rotation by 8 inside the row, a
// data-parallel-primitive operand modifier, no LDS round trip)
__device__ __forceinline__ float lane_xor8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128 /* row_ror:8 */, 0xf, 0xf, false));
}

__device__ __forceinline__ int lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// ---- global memory -> LDS without passing through registers (global_load_lds).  Every lane
// gives a byte offset from a wave-uniform base address; the 64 chunks of a wave land next to
// each other from the wave-uniform LDS address on (lane * 16 or lane * 4 bytes in).
// Written as inline assembly on purpose: when the compiler knows of such a load it makes every
// later LDS read wait for all of them, which would undo the prefetching.  The loads complete
// in order and are counted by vmcnt, so "all but the n youngest have landed" is wait_vmcnt<n>;
// loads the compiler issues itself in between only make that wait longer, never shorter.
// (m0 is reserved: the compiler sets it immediately before each of its own uses.  The s_nop is
// the wait state between a scalar write of m0 and a memory instruction that reads it; inside
// inline assembly nobody else would insert it.)
__device__ __forceinline__ uint32_t lds_addr(const void* p)
{
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t byte_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(byte_off), "s"(base) : "memory");
}
// the same marked non-temporal: rows that nobody else will ask for (a list scanned by one work item) should not
// push the rows that several work items share out of the L2
__device__ __forceinline__ void lds_dma16_nt(const void* base, uint32_t byte_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" :: "s"(lds), "v"(byte_off), "s"(base) : "memory");
}
__device__ __forceinline__ void lds_dma4(const void* base, uint32_t byte_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(lds), "v"(byte_off), "s"(base) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// inclusive prefix sum over the 64 lanes of a wave (row shifts inside each group of 16 lanes,
// then the last lane of rows 0..2 added to the rows after it)
__device__ __forceinline__ int wave_prefix_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v;
}

// sum over the 64 lanes of a wave, in the last lane (the lane steps of the prefix sum above)
__device__ __forceinline__ float wave_add(float v)
{
    auto from = [&](auto step, auto rows) __attribute__((always_inline)) {
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(step)::value, decltype(rows)::value, 0xf, false));
    };
    using std::integral_constant;
    from(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
    from(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    from(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    from(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    from(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    from(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
    return v;
}

// bitwise or / smallest value over the 64 lanes of a wave, to all lanes (the lane steps of the prefix sum above; lanes
// that a step does not reach combine their value with itself)
template <typename F>
__device__ __forceinline__ uint32_t wave_fold(uint32_t v, F&& f)
{
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xf, 0xf, false));
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xf, 0xf, false));
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xf, 0xf, false));
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xf, 0xf, false));
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));
    v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) { return wave_fold(v, [](uint32_t x, uint32_t y) { return x | y; }); }
__device__ __forceinline__ uint32_t wave_min(uint32_t v) { return wave_fold(v, [](uint32_t x, uint32_t y) { return x < y ? x : y; }); }

// largest of 64 numbers, none of them negative (their bits are in order)
__device__ __forceinline__ float wave_max(float v)
{
    return __builtin_bit_cast(float, wave_fold(__builtin_bit_cast(uint32_t, v), [](uint32_t x, uint32_t y) { return x > y ? x : y; }));
}

}  // namespace hr
