// What the general kernels (fp32, and bf16 with channel counts outside the wide matrix tiles) share:
// the fp32 matrix instruction, and four consecutive channels as one access.
#pragma once
#include "common.h"

namespace k3 {

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// four / one values at element offset off (negative: zero) behind a descriptor, plus soff bytes
template <typename T> struct buf;
template <> struct buf<float> {
    static __device__ __forceinline__ f32x4 quad(__amdgpu_buffer_rsrc_t r, int off, int soff)
    {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off < 0 ? -1 : off * 4, soff, 0));
    }
    static __device__ __forceinline__ float one(__amdgpu_buffer_rsrc_t r, int off, int soff)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off < 0 ? -1 : off * 4, soff, 0));
    }
    static __device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
    static __device__ __forceinline__ void st4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
};
template <> struct buf<bf16_t> {
    static __device__ __forceinline__ f32x4 wide(uint2 v)
    {
        return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
    }
    static __device__ __forceinline__ f32x4 quad(__amdgpu_buffer_rsrc_t r, int off, int soff)
    {
        return wide(__builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off < 0 ? -1 : off * 2, soff, 0)));
    }
    static __device__ __forceinline__ float one(__amdgpu_buffer_rsrc_t r, int off, int soff)
    {
        return bf2f((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off < 0 ? -1 : off * 2, soff, 0));
    }
    static __device__ __forceinline__ f32x4 ld4(const bf16_t *p) { return wide(*reinterpret_cast<const uint2 *>(p)); }
    static __device__ __forceinline__ void st4(bf16_t *p, f32x4 v)
    {
        *reinterpret_cast<uint2 *>(p) = make_uint2(pack2bf(v[0], v[1]), pack2bf(v[2], v[3]));
    }
};

__device__ __forceinline__ f32x4 keep_positive(f32x4 v, f32x4 m)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = m[j] > 0.f ? v[j] : 0.f;
    return v;
}

// A lane group kg of 16 lanes holds values 4 kg .. 4 kg + 3 of 16; afterwards v[j] holds value 4 j + kg: the
// operands of four instructions in the order of the values (a 4 x 4 transposition over the lane groups).
__device__ __forceinline__ void spread(float (&v)[4])
{
    auto swap32 = [](float &a, float &b) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    auto swap16 = [](float &a, float &b) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    swap32(v[0], v[2]);
    swap32(v[1], v[3]);
    swap16(v[0], v[1]);
    swap16(v[2], v[3]);
}

}  // namespace k3
