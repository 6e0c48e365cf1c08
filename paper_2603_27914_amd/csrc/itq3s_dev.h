// Device-side helpers shared by the libitq3s kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace itq3s {

constexpr int kBlock = 256;        // elements per quantization block (the transform length)
constexpr int kTileRows = 16;      // rows per storage tile
constexpr int kTileWords = 384;    // uint32 per tile: 256 low-plane + 128 high-plane
constexpr int kTileLoWords = 256;
constexpr int kWave = 64;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

__device__ __forceinline__ float f16_bits_to_f32(uint32_t bits16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// Cross-lane exchange with lane (l ^ mask), 32-bit payload.
__device__ __forceinline__ int xor_lane_i32(int v, int mask) { return __shfl_xor(v, mask, 64); }
__device__ __forceinline__ float xor_lane_f32(float v, int mask) { return __shfl_xor(v, mask, 64); }
__device__ __forceinline__ double xor_lane_f64(double v, int mask) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_xor(lo, mask, 64);
    hi = __shfl_xor(hi, mask, 64);
    return __hiloint2double(hi, lo);
}

// value of lane (l ^ MASK), MASK < 32, through the LDS crossbar (ds_swizzle in bit-mask mode: no
// memory access).  One instruction per 32 bits for any distance, and it runs beside the vector ALU
// rather than on it -- data-parallel-primitive moves need two per distance 4 or 8 and measured 12 %
// slower in the fp64 butterfly kernels, which are bound by vector-ALU issue.
template <int MASK>
__device__ __forceinline__ int row_xor_i32(int x) {
    return __builtin_amdgcn_ds_swizzle(x, (MASK << 10) | 0x1F);
}
template <int MASK>
__device__ __forceinline__ double row_xor_f64(double v) {
    const int lo = row_xor_i32<MASK>(__double2loint(v)), hi = row_xor_i32<MASK>(__double2hiint(v));
    return __hiloint2double(hi, lo);
}

// H_16[4g + j][r16] / 4, j = 0..3: B operand of the first product, A operand of the second.  The sign of an
// entry is the parity of (4g + j) & r16: that of 4g & r16, flipped for j = 1, 3 by bit 0 of r16 and for
// j = 2, 3 by bit 1.
__device__ __forceinline__ half4 hadamard_quarter(int lane) {
    const uint32_t r = (uint32_t)lane & 15u, g = (uint32_t)lane >> 4;
    const uint32_t s = (g & (r >> 2)) ^ ((g >> 1) & (r >> 3));
    const uint32_t lo = ((s & 1u) << 15) | (((s ^ r) & 1u) << 31);
    const uint32_t w0 = 0x34003400u ^ lo, w1 = w0 ^ ((r >> 1) & 1u) * 0x80008000u;
    return __builtin_bit_cast(half4, u32x2{w0, w1});
}

// fp4 operands of the block-scaled products: the codes c of a low-plane word's even slots (bits 1:0 of its nibbles) and
// of its odd slots (bits 3:2), as c / 2 (0, 0.5, 1, and 1.5 for a 3: the format's one linear run of codes, so the odd ones
// take a shift more than they would as 2, 0, -2); and the scales of B that go with them and the three parts of A (bytes
// 0..2: 2^(1, -3, -8)).
__device__ __forceinline__ uint32_t even_digits(uint32_t v) { return v & 0x33333333u; }
__device__ __forceinline__ uint32_t odd_digits(uint32_t v) { return (v >> 2) & 0x33333333u; }
constexpr int kDigitScales = 0x00777c80;

// Groups of 32 activations that are fp16 (rotate_mx_kernel says which and why) have a scale of 0, which none has otherwise
// and which takes what their bytes are as fp6 to below 1e-35.  Of a lane's four scales: bit 8 q + 7 for step q.
__device__ __forceinline__ uint32_t wide_steps(uint32_t scales) { return (scales - 0x01010101u) & ~scales & 0x80808080u; }

}  // namespace itq3s
