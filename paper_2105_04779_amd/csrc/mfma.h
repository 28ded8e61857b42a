// What the kernels on the 16-bit matrix instructions share: operand types, the instructions, reductions inside 16 lanes.
#pragma once
#include "el_internal.h"

namespace el {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
#define EL_LDS(T) __attribute__((address_space(3))) T

constexpr int kTile = 16;                 // rows of H per tile
constexpr float kMasked = -1.0e30f;       // score of a position that does not exist: finite, exp2 of it is 0

template <bool BF16> struct Mma;
template <> struct Mma<false> {
    static __device__ __forceinline__ f4 s16(u4 a, u4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0); }
    static __device__ __forceinline__ f16v s32(u4 a, u4 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0); }
};
template <> struct Mma<true> {
    static __device__ __forceinline__ f4 s16(u4 a, u4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0); }
    static __device__ __forceinline__ f16v s32(u4 a, u4 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0); }
};

// x = high + low, both in the 16-bit storage type, of two neighbours at once (split16 with the conversion instruction that rounds a
// pair to bf16: three instructions a value instead of some twenty).  A NaN stays one.
template <bool BF16>
__device__ __forceinline__ void split16_pair(float x, float y, unsigned &high, unsigned &low)
{
    if (BF16) {
        high = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{x, y}, b2));
        low = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{x - __uint_as_float(high << 16), y - __uint_as_float(high & 0xffff0000u)}, b2));
    } else {
        const h2 h = __builtin_convertvector(f2{x, y}, h2);
        high = __builtin_bit_cast(unsigned, h);
        low = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{x - (float)h[0], y - (float)h[1]}, h2));
    }
}

// a value of another lane of the same 16 on the vector ALU (DPP), no LDS round trip
template <int CTRL> __device__ __forceinline__ float dpp(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true)); }
__device__ __forceinline__ float quad_xor1(float v) { return dpp<0xB1>(v); }
__device__ __forceinline__ float quad_xor2(float v) { return dpp<0x4E>(v); }
__device__ __forceinline__ float dpp_half_mirror(float v) { return dpp<0x141>(v); }     // lane i <-> 7 - i of each 8
__device__ __forceinline__ float dpp_row_mirror(float v) { return dpp<0x140>(v); }      // lane i <-> 15 - i of each 16
__device__ __forceinline__ float max16(float v)
{
    v = fmaxf(v, quad_xor1(v)); v = fmaxf(v, quad_xor2(v)); v = fmaxf(v, dpp_half_mirror(v));
    return fmaxf(v, dpp_row_mirror(v));
}
__device__ __forceinline__ float sum16(float v)
{
    v += quad_xor1(v); v += quad_xor2(v); v += dpp_half_mirror(v);
    return v + dpp_row_mirror(v);
}

} // namespace el
