// Weight-side reconstruction (Alg. 2, Prop. 1): w_hat = H( d (q - z) ).
//
// q takes small integer values, so the transform of the digits is exact in any arithmetic that holds
// integers up to 512; the zero-point only reaches element 0 (H applied to a constant vector is a
// spike: H 1 = 16 e_0) and is folded in after the transform.  One rounding per output element.
//
// The 256-point transform runs on the matrix cores.  With the block written as a 16 x 16 matrix
// V[a][b] = v[16a + b], the Sylvester construction gives H_256 = H_16 (x) H_16, so
// (H_u v)[16a' + b'] = (H_16 V H_16)[a'][b'] with the +-1 matrix H_16.  The kernel forms the
// transpose, U^T = H_16 (V^T H_16): two 16x16x16 products on fp16 inputs (digits, then integers up
// to 32: all exact) with fp32 sums.  The accumulator layout of the first product is the B-operand
// layout of the second, and the transposed result leaves every lane with four consecutive output
// elements, e = 16 (l%16) + 4 (l/16) + 0..3: a wavefront stores one contiguous row segment.
//
// What bounds it: the stores (2 or 4 bytes per weight against 0.39 read).  A wavefront takes eight or four rows of a
// 16-row tile: it loads the tile's words once, coalesced (its lane of the rows' operand layout: 16 + 8 + 4
// bytes), and hands a row's words to the lanes that need them inside the 16-lane rows of the vector ALU.
// (Loading every row's words where they are needed -- four different addresses per instruction, twelve
// instructions per four rows -- kept the address units busy for half of the launch.)  For fp16 output two rows
// exchange halves between neighbouring 16-lane rows, so that a lane stores 16 bytes; the stores carry the
// nontemporal hint (28672x8192 fp16 101 -> 78 us, fp32 180 -> 144).  Before / now, us, several outputs in turn:
// 11008x4096 fp16 31.6 / 16.6, 28672x8192 fp16 152 / 78 (7.2 TB/s in all), fp32 207 / 144.
#include <type_traits>

#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

// Sixteen bytes that promise the alignment of eight: ldo need only be a multiple of four elements, so rows of
// fp16 output may start between two 16-byte boundaries.
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

// Rows per wavefront.  fp32: four -- with eight, 11008x4096 took 34 us instead of 30 and 28672x8192 171 instead
// of 144 (more rows of one wavefront open at a time).  fp16: eight (28672x8192 84 us with four, 78 with eight;
// 4096x4096 8.1 and 7.4), but four for up to 1024 tiles: all wavefronts are resident at once then, and what
// counts is the length of one (4096x256 3.76 us with eight, 3.47 with four; 1000x4096 4.50 and 4.31, 2048x4096,
// which is beyond, 5.17 and 5.29).
constexpr int64_t kDqShortTiles = 1024;  // 4096 wavefronts of four rows: four per SIMD

// value of lane R of the lane's own 16-lane row
template <int R>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + R, 0xf, 0xf, true);
}
template <int R>
__device__ __forceinline__ float row_lane(float v) {
    return __builtin_bit_cast(float, row_lane<R>(__builtin_bit_cast(uint32_t, v)));
}

// kSub: the sub-block-scale variant (Sec. 4.1: 116 bytes per block), w_hat = H( d (s_j q - z) ).  A lane's
// four digits belong to sub-blocks 2g (the first two) and 2g+1, whose scales are the two halves of
// the lane's own word of the sub-scale array; s q is exact in fp16, the first product (16 terms of one
// sub-block: a 16-bit number) is carried in two fp16 parts, the second adds 16 such terms in fp32.
struct DqTile {  // a lane's words of the wavefront's rows: storage lane 16 g + row of the tile for r16 = row - first row
    u32x4 lo;
    u32x2 hi;
    uint32_t ss;
    float d16, z256;  // d / 16 (exact: one rounding per output) and 256 z of row r16
};

// Row R (0..7) of the wavefront: elements 16 r16 + 4 g + 0..3 of its block, not yet rounded to the output type.
template <int R, bool kSub>
__device__ __forceinline__ floatx4 dequantize_row(const DqTile& t, bool any_hi, const half4& h, int lane) {
    // elements e = 64 g + 16 j + r16 (j = 0..3) sit in slot r16 of low-plane word j of storage lane 16 g + r;
    // their high bits in bit 16 (j & 1) + r16 of high-plane word j >> 1
    const int r16 = lane & 15;
    const uint32_t sh = 2u * (uint32_t)r16;
    const uint32_t c0 = __builtin_amdgcn_ubfe(row_lane<R>(t.lo.x), sh, 2u), c1 = __builtin_amdgcn_ubfe(row_lane<R>(t.lo.y), sh, 2u);
    const uint32_t c2 = __builtin_amdgcn_ubfe(row_lane<R>(t.lo.z), sh, 2u), c3 = __builtin_amdgcn_ubfe(row_lane<R>(t.lo.w), sh, 2u);
    uint32_t p01 = c0 | (c1 << 16), p23 = c2 | (c3 << 16);
    if (any_hi) {  // (malformed input only; uniform) the high bits count 4: the digit is still code - 1
        const uint32_t hx = row_lane<R>(t.hi.x), hy = row_lane<R>(t.hi.y);
        p01 |= (((hx >> r16) & 1u) << 2) | (((hx >> (16 + r16)) & 1u) << 18);
        p23 |= (((hy >> r16) & 1u) << 2) | (((hy >> (16 + r16)) & 1u) << 18);
    }
    // OR-ed into the mantissa of the half 1024.0, whose lowest mantissa bit weighs exactly 1: 1024 + c,
    // minus 1025, is the digit c - 1 (exact)
    const half2v bias = {(_Float16)(-1025.0f), (_Float16)(-1025.0f)};
    const half2v v01 = __builtin_bit_cast(half2v, p01 | 0x64006400u) + bias, v23 = __builtin_bit_cast(half2v, p23 | 0x64006400u) + bias;
    half4 v = {v01[0], v01[1], v23[0], v23[1]};
    if constexpr (kSub) {
        const half2v s2 = __builtin_bit_cast(half2v, row_lane<R>(t.ss));
        v = half4{v[0] * s2[0], v[1] * s2[0], v[2] * s2[1], v[3] * s2[1]};
    }
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    const floatx4 T = __builtin_amdgcn_mfma_f32_16x16x16f16(v, h, zero, 0, 0, 0);  // V^T H_16, |.| <= 16 * 6
    const half4 th = __builtin_convertvector(T, half4);
    floatx4 U = __builtin_amdgcn_mfma_f32_16x16x16f16(h, th, zero, 0, 0, 0);
    if constexpr (kSub) {
        floatx4 rest;
#pragma unroll
        for (int i = 0; i < 4; ++i) rest[i] = __builtin_fmaf((float)th[i], -1.0f, T[i]);  // exact
        U = __builtin_amdgcn_mfma_f32_16x16x16f16(h, __builtin_convertvector(rest, half4), U, 0, 0, 0);
    }
    const float d16 = row_lane<R>(t.d16), z256 = row_lane<R>(t.z256);
    U[0] = U[0] - (lane == 0 ? z256 : 0.0f);  // H_u applied to the constant -z reaches element 0 only
    return floatx4{d16 * U[0], d16 * U[1], d16 * U[2], d16 * U[3]};
}

template <bool kOutF16, bool kSub, int kRows>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void dequantize_kernel(const uint32_t* __restrict__ codes, const uint32_t* __restrict__ scales,
                                                         const uint32_t* __restrict__ subscales, int64_t N, int KB, int64_t parts, void* __restrict__ out, int64_t ldo,
                                                         uint32_t* __restrict__ flags) {
    const int lane = lane_id();
    const int64_t part = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // kParts per tile
    if (part >= parts) return;
    constexpr int kParts = kTileRows / kRows;
    const uint32_t tile = (uint32_t)(part / kParts), nt = tile / (uint32_t)KB, b = tile - nt * (uint32_t)KB;
    const int first = (int)(part % kParts) * kRows;
    const int r16 = lane & 15, g = lane >> 4;
    const int row = (first + r16) & 15;  // of the tile: the wavefront's rows are those of r16 < kRows
    const uint32_t* const t = codes + (int64_t)tile * kTileWords;
    DqTile w;
    w.lo = *reinterpret_cast<const u32x4*>(t + 4 * (16 * g + row));
    w.hi = *reinterpret_cast<const u32x2*>(t + kTileLoWords + 2 * (16 * g + row));
    const uint32_t sw = scales[(int64_t)tile * kTileRows + row];
    w.ss = kSub ? subscales[(int64_t)tile * 64 + 16 * g + row] : 0u;

    half4 h;  // H_16[4g + j][r16]: B operand of the first product, A operand of the second
    {
        const half4 q = hadamard_quarter(lane);
        h = half4{q[0] * (_Float16)4.0f, q[1] * (_Float16)4.0f, q[2] * (_Float16)4.0f, q[3] * (_Float16)4.0f};
    }
    w.d16 = f16_bits_to_f32(sw & 0xffffu) * 0.0625f;
    w.z256 = f16_bits_to_f32(sw >> 16) * 256.0f;
    // a code 3 in the low plane, or any bit of the high plane, is a format error (every wavefront
    // of a tile looks at all of its rows)
    const uint32_t three = ((w.lo.x & (w.lo.x >> 1)) | (w.lo.y & (w.lo.y >> 1)) | (w.lo.z & (w.lo.z >> 1)) | (w.lo.w & (w.lo.w >> 1))) & 0x55555555u;
    const bool any_hi = __builtin_amdgcn_ballot_w64((w.hi.x | w.hi.y) != 0u) != 0ull;
    if (flags != nullptr && __builtin_amdgcn_ballot_w64((three | w.hi.x | w.hi.y) != 0u) != 0ull && lane == 0) atomicOr(flags, kFlagBadCode);

    const int64_t n0 = (int64_t)nt * kTileRows + first;  // (rows past N exist in storage; only their store is skipped)
    const int64_t col = (int64_t)b * kBlock;
    auto pair = [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        const floatx4 f0 = dequantize_row<R, kSub>(w, any_hi, h, lane), f1 = dequantize_row<R + 1, kSub>(w, any_hi, h, lane);
        if constexpr (kOutF16) {
            u32x2 a = __builtin_bit_cast(u32x2, __builtin_convertvector(f0, half4)), c = __builtin_bit_cast(u32x2, __builtin_convertvector(f1, half4));
            // 16-lane rows 0, 2 keep row R and 1, 3 row R + 1: elements 16 r16 + 8 (g / 2) + 0..7
            const auto s0 = __builtin_amdgcn_permlane16_swap(a.x, c.x, false, false), s1 = __builtin_amdgcn_permlane16_swap(a.y, c.y, false, false);
            const int64_t n = n0 + R + (g & 1);
            if (n < N)
                __builtin_nontemporal_store(u32x4_a8{s0[0], s1[0], s0[1], s1[1]},
                                            reinterpret_cast<u32x4_a8*>(reinterpret_cast<_Float16*>(out) + n * ldo + col + 16 * r16 + 8 * (g >> 1)));
        } else {
            float* const dst = reinterpret_cast<float*>(out) + (n0 + R) * ldo + col + 16 * r16 + 4 * g;
            if (n0 + R < N) __builtin_nontemporal_store(f0, reinterpret_cast<floatx4*>(dst));
            if (n0 + R + 1 < N) __builtin_nontemporal_store(f1, reinterpret_cast<floatx4*>(dst + ldo));
        }
    };
    pair(std::integral_constant<int, 0>{});
    pair(std::integral_constant<int, 2>{});
    if constexpr (kRows == 8) {
        pair(std::integral_constant<int, 4>{});
        pair(std::integral_constant<int, 6>{});
    }
}

template <bool kOutF16, int kRows>
static int launch_dequantize_rows(const uint32_t* codes, const uint32_t* scales, const uint32_t* subscales, int64_t N, int64_t tiles, int KB, void* out,
                                  int64_t ldo, uint32_t* flags, hipStream_t stream) {
    const int64_t parts = tiles * (kTileRows / kRows);
    const dim3 grid((unsigned)((parts + 3) / 4)), block(256);
    if (subscales != nullptr) hipLaunchKernelGGL((dequantize_kernel<kOutF16, true, kRows>), grid, block, 0, stream, codes, scales, subscales, N, KB, parts, out, ldo, flags);
    else hipLaunchKernelGGL((dequantize_kernel<kOutF16, false, kRows>), grid, block, 0, stream, codes, scales, subscales, N, KB, parts, out, ldo, flags);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

int launch_dequantize(const uint32_t* codes, const uint32_t* scales, const uint32_t* subscales, int64_t N, int64_t K, void* out, int out_f16,
                      int64_t ldo, uint32_t* flags, hipStream_t stream) {
    const int64_t tiles = ((N + 15) / 16) * (K / kBlock);
    const int KB = (int)(K / kBlock);
    if (!out_f16) return launch_dequantize_rows<false, 4>(codes, scales, subscales, N, tiles, KB, out, ldo, flags, stream);
    if (tiles <= kDqShortTiles) return launch_dequantize_rows<true, 4>(codes, scales, subscales, N, tiles, KB, out, ldo, flags, stream);
    return launch_dequantize_rows<true, 8>(codes, scales, subscales, N, tiles, KB, out, ldo, flags, stream);
}

}  // namespace itq3s
