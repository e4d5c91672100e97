// Device helpers of the register-streamed kernels (hpsi_rs64.hip, hpsi_big64.hip, hpsi_lds.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace dmrg {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// wave-uniform values in scalar registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double unid(double v) {
    return __builtin_bit_cast(double, uni64(__builtin_bit_cast(int64_t, v)));
}

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ..: a loop whose indices are constants before
// any optimisation. As an unrolled loop, an array of accumulators becomes one vector register of 16 .. 64
// dwords first, and every conditional MFMA copies all of it.
template <class F, int... I>
__device__ __forceinline__ void each_of(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(F&& f) {
    each_of(f, std::make_integer_sequence<int, N>{});
}

// keeps the loads before it from sinking to their uses and those after it from rising
__device__ __forceinline__ void fence() { asm volatile("" ::: "memory"); }

// `bytes` at p for buffer loads; what a load asks for past them is zero and moves nothing. The card checks the sum of
// the lane's and the scalar offset (4096 bytes and 0 .. 65536 as the scalar offset: zeros from 4096 on); by the
// intrinsic's contract alone it is the lane's offset, hence kOperandSlack (internal.h).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00027000);
}
// 16 bytes at byte lane_bytes + at (wave-uniform, the scalar offset)
__device__ __forceinline__ i32x4 ld16(__amdgpu_buffer_rsrc_t b, uint32_t lane_bytes, uint32_t at) {
    return (i32x4)__builtin_amdgcn_raw_buffer_load_b128(b, (int)lane_bytes, (int)at, 0);
}

// An offset outside every buffer (also with a small constant added)
constexpr uint32_t kNowhere = 0x80000000u;

// ---------------------------------------------------------------- split BF16 operands
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Frag { u16x8 h, l; };   // a lane's part of a 16 x 32 tile, hi and lo
// tile at byte lane_bytes + at: 1 KB of hi parts in lane order, then 1 KB of lo parts
__device__ __forceinline__ Frag ld_frag(__amdgpu_buffer_rsrc_t b, uint32_t lane_bytes, uint32_t at = 0) {
    return Frag{__builtin_bit_cast(u16x8, ld16(b, lane_bytes, at)), __builtin_bit_cast(u16x8, ld16(b, lane_bytes + 1024u, at))};
}
// product W of a.b: hi hi, hi lo, lo hi
template <int W>
__device__ __forceinline__ f32x4 mma(const Frag& a, const Frag& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W < 2 ? a.h : a.l),
                                                   __builtin_bit_cast(bf16x8, W == 1 ? b.l : b.h), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
// hi and lo parts of eight products f x (v_cvt_pk_bf16_f32 rounds two at a time to nearest even)
__device__ __forceinline__ Frag split8(float f, const float (&x)[8]) {
    u32x4 h, l;
    each<4>([&](auto i) {
        constexpr int k = i;
        h[k] = pack2(f * x[2 * k], f * x[2 * k + 1]);
        l[k] = pack2(__builtin_fmaf(f, x[2 * k], -__builtin_bit_cast(float, h[k] << 16)),
                     __builtin_fmaf(f, x[2 * k + 1], -__builtin_bit_cast(float, h[k] & 0xffff0000u)));
    });
    return Frag{__builtin_bit_cast(u16x8, h), __builtin_bit_cast(u16x8, l)};
}

}  // namespace dmrg
