// Activation-side rotation.  H is symmetric and its own inverse (Sec. 2.3), hence
//   <H v, x> = <v, H x>:
// instead of transforming every weight block, each 256-channel chunk of the activations is
// transformed once per call and the ternary digits are contracted with the rotated chunk.
//
// One wavefront per (row m, chunk b).  The 256-point transform runs on the matrix cores: with the
// chunk written as a 16 x 16 matrix X[a][b] = x[16a + b], the Sylvester construction gives
// H_256 = H_16 (x) H_16, i.e. (H x)[16a' + b'] = (H_16 X H_16)[a'][b'] / 16 (H_16 with entries +-1).
// T = X (H_16/4) is one 16x16x16 product (fp16 inputs, exact products, fp32 sums; the factor keeps
// |T| <= 4 max|x| inside the fp16 range); H_16 T follows with T split into two halves
// (T = T_hi + T_lo keeps 22 bits), then the remaining factor 1/4 and one rounding to fp16.  The
// accumulator layout of the first product is the B-operand layout of the second, so nothing moves
// between lanes.
#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

// x~ = H x for one chunk.  Lane l reads x[16 (l%16) + 4 (l/16) + 0..3] and returns the rounded
// elements e = 64 (l/16) + 16 i + l%16, i = 0..3.
// Returns false if a rotated value (or the intermediate T, which then turns the result into NaN)
// leaves the fp16 range.
__device__ __forceinline__ bool rotate_operand(half4 xa, int lane, _Float16 out[4]) {
    const half4 q = hadamard_quarter(lane);
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    const floatx4 T = __builtin_amdgcn_mfma_f32_16x16x16f16(xa, q, zero, 0, 0, 0);
    const half4 th = __builtin_convertvector(T, half4);
    floatx4 rest;
#pragma unroll
    for (int j = 0; j < 4; ++j) rest[j] = __builtin_fmaf((float)th[j], -1.0f, T[j]);  // exact
    const half4 tl = __builtin_convertvector(rest, half4);
    floatx4 U = __builtin_amdgcn_mfma_f32_16x16x16f16(q, th, zero, 0, 0, 0);
    U = __builtin_amdgcn_mfma_f32_16x16x16f16(q, tl, U, 0, 0, 0);
    const half4 r = __builtin_convertvector(U, half4);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = r[i];
    // (a maximum that hands a NaN on)
    const float peak = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(U[0]), __builtin_fabsf(U[1])),
                                                     __builtin_elementwise_maximum(__builtin_fabsf(U[2]), __builtin_fabsf(U[3])));
    return peak <= 65504.0f;
}

// The same from memory.  `first` receives the first of the lane's four inputs (lane 0: x[0]).
__device__ __forceinline__ bool rotate_chunk(const _Float16* __restrict__ src, int lane, _Float16 out[4], _Float16* first = nullptr) {
    const half4 xa = *reinterpret_cast<const half4*>(src + 16 * (lane & 15) + 4 * (lane >> 4));
    if (first != nullptr) *first = xa[0];
    return rotate_operand(xa, lane, out);
}

// Operand order of the streaming kernel.  The 16x16x32 MFMA of step t (0..7) takes from lane
// (column m, k-group g) eight halves; position i of those eight is element
//     e = 64 g + 16 (t>>1) + 4 (t&1) + (i>>1) + 8 (i&1)
// of the chunk, which is where the weight kernel's shift-and-mask unpack puts the code of the same
// element.  Xt index = (((b*8 + t)*4 + g)*MP + m)*8 + i.   S[b*MP + m] = sum_e x~_e (rounded values),
// S[KB*MP + b*MP + m] = 16 x_0 (the same sum before rounding, exact).
// (at least two wavefronts per SIMD: with a register budget of 256 the matrix instructions write ordinary
// vector registers; with the full 512 the compiler parks their results in accumulator registers and copies
// every one of them out)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void rotate_frag_kernel(const _Float16* __restrict__ X, int64_t M, int64_t K, int64_t ldx, int MP,
                                                          _Float16* __restrict__ Xt, float* __restrict__ S, uint32_t* __restrict__ flags) {
    const int KB = (int)(K / kBlock);
    const int lane = lane_id();
    // (32-bit, wave-uniform index arithmetic: MP * KB chunks, far below 2^31)
    const int chunk = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // m * KB + b over MP rows
    if (chunk >= MP * KB) return;
    const int m = chunk / KB, b = chunk - m * KB;
    _Float16 r[4] = {(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
    _Float16 x0 = (_Float16)0.f;
    if (m < M && !rotate_chunk(X + (int64_t)m * ldx + (int64_t)b * kBlock, lane, r, &x0) && flags != nullptr) atomicOr(flags, kFlagActRange);
    // sum of the rounded chunk: inside a row of 16 lanes through the crossbar, the four rows through scalar registers
    float s = ((float)r[0] + (float)r[1]) + ((float)r[2] + (float)r[3]);
    s += __builtin_bit_cast(float, row_xor_i32<1>(__builtin_bit_cast(int, s)));
    s += __builtin_bit_cast(float, row_xor_i32<2>(__builtin_bit_cast(int, s)));
    s += __builtin_bit_cast(float, row_xor_i32<4>(__builtin_bit_cast(int, s)));
    s += __builtin_bit_cast(float, row_xor_i32<8>(__builtin_bit_cast(int, s)));
    const float total = (__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 0)) +
                         __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 16))) +
                        (__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 32)) +
                         __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 48)));
    if (lane == 0) {
        S[b * MP + m] = total;
        // exact sum of the unrounded chunk: H 1 = 16 e_0 (lane 0 holds x[0] from its operand load)
        S[KB * MP + b * MP + m] = 16.0f * (float)x0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int e = 64 * (lane >> 4) + 16 * j + (lane & 15);
        const int g = e >> 6, w = (e >> 4) & 3, slot = e & 15;
        const int t = 2 * w + ((slot & 7) >> 2);
        const int i = 2 * (slot & 3) + (slot >> 3);
        Xt[(((((int64_t)b * 8 + t) * 4 + g) * MP + m) * 8) + i] = r[j];
    }
}

// Operand order of the streaming kernel for 17 and more rows (itq3s_rows.hip): rows in groups of 16 mt, a
// group's fragments (t, mt) of a block one after another, 1 KiB each -- lane l = 16 g + r of the MFMA
// operand finds its eight halves, the same elements as above, at 16 l.
//   Xt index = ((((group*KB + b)*8 + t)*mts + mt)*64 + l)*8 + i,   row m = (group*mts + mt)*16 + r
//   X0 index = ((group*KB + b)*4 + q)*stride + 4 mt + i = x[(group*mts + mt)*16 + 4 q + i][256 b], stride 8 for
//              mts <= 2, else 16
// Rows past M are zero.  A workgroup rotates 16 rows of one block, two per wavefront, and passes the
// rounded values through LDS (rows in the channel order in which a lane's eight halves are neighbours),
// so that every store is 16 bytes and a wavefront's are 1 KiB of consecutive addresses.
constexpr int kRotRowStride = 264;  // halves; 528 bytes: 16-byte reads of 16 rows touch all banks
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void rotate_rows_kernel(const _Float16* __restrict__ X, int M, int KB, int64_t ldx, int mts,
                                                              _Float16* __restrict__ Xt, _Float16* __restrict__ X0, uint32_t* __restrict__ flags) {
    __shared__ __align__(16) _Float16 rows[16 * kRotRowStride];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tile = (int)blockIdx.x / KB, b = (int)blockIdx.x - tile * KB;  // tile = group * mts + mt
    const int group = tile / mts, mt = tile - group * mts;
    half4 xa[2];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        const int m = tile * 16 + wave * 2 + rr;
        xa[rr] = half4{(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
        if (m < M) xa[rr] = *reinterpret_cast<const half4*>(X + (int64_t)m * ldx + (int64_t)b * kBlock + 16 * (lane & 15) + 4 * (lane >> 4));
    }
    bool ok = true;
    const int s = lane & 15;
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        _Float16 r[4];
        ok = rotate_operand(xa[rr], lane, r) && ok;
        _Float16* const dst = rows + (wave * 2 + rr) * kRotRowStride + 64 * (lane >> 4) + 2 * (s & 7) + (s >> 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[16 * j] = r[j];
    }
    const int64_t gb = (int64_t)group * KB + b;
    if (lane == 0) *reinterpret_cast<half2v*>(X0 + (gb * 4 + (wave >> 1)) * (mts <= 2 ? 8 : 16) + 4 * mt + 2 * (wave & 1)) = half2v{xa[0][0], xa[1][0]};
    if (!ok && flags != nullptr) atomicOr(flags, kFlagActRange);
    __syncthreads();
    const u32x4 v = *reinterpret_cast<const u32x4*>(rows + (lane & 15) * kRotRowStride + 64 * (lane >> 4) + 16 * (wave >> 1) + 8 * (wave & 1));
    *reinterpret_cast<u32x4*>(Xt + (((gb * 8 + wave) * mts + mt) * 64 + lane) * 8) = v;  // step t = wave
}

// Operand order of the tiled kernel: rows stay rows; inside every group of 16 channels, slot s moves
// to position 2 (s & 7) + (s >> 3), the order in which the tile loader's unpack emits the weights.
// A wavefront rotates four consecutive chunks (of the list row by row), loads first, and passes the rounded
// values through a corner of LDS of its own, so that it stores 1 KiB of consecutive addresses per
// instruction: bound by memory, not by the number of 2-byte stores (2048 x 14336: 31 -> 24 us, at the
// 5.1 TB/s of a large copy).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void rotate_rowmajor_kernel(const _Float16* __restrict__ X, int64_t chunks, int KB, int64_t ldx,
                                                              _Float16* __restrict__ Xt, uint32_t* __restrict__ zero_words, int n_zero, uint32_t* __restrict__ flags) {
    __shared__ __align__(16) _Float16 lds[4][4 * kBlock];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // the split-K flags of the contraction that follows start from zero
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_zero; i += 256) zero_words[i] = 0u;
    const int64_t first = ((int64_t)blockIdx.x * 4 + wave) * 4;
    const int n = chunks - first < 4 ? (int)(chunks - first) : 4;
    if (n <= 0) return;
    half4 xa[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t chunk = (uint32_t)(first + (c < n ? c : 0)), m = chunk / (uint32_t)KB, b = chunk - m * (uint32_t)KB;  // (M K / 256 is below 2^31)
        xa[c] = *reinterpret_cast<const half4*>(X + (int64_t)m * ldx + (int64_t)b * kBlock + 16 * (lane & 15) + 4 * (lane >> 4));
    }
    const int s = lane & 15;
    bool ok = true;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        _Float16 r[4];
        ok = rotate_operand(xa[c], lane, r) && ok;
        _Float16* const dst = lds[wave] + c * kBlock + 64 * (lane >> 4) + 2 * (s & 7) + (s >> 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[16 * j] = r[j];
    }
    if (!ok && flags != nullptr) atomicOr(flags, kFlagActRange);
    // (one wavefront writes and reads: the LDS instructions of a wavefront stay in order)
    __builtin_amdgcn_wave_barrier();
    u32x4* const out = reinterpret_cast<u32x4*>(Xt + first * kBlock);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(lds[wave] + (64 * u + lane) * 8);
        if (2 * u + (lane >> 5) < n) out[64 * u + lane] = v;
    }
}

int launch_rotate_frag(const _Float16* X, int64_t M, int64_t K, int64_t ldx, int MP, _Float16* Xt, float* S, uint32_t* flags, hipStream_t stream) {
    const int64_t chunks = (int64_t)MP * (K / kBlock);
    hipLaunchKernelGGL(rotate_frag_kernel, dim3((unsigned)((chunks + 3) / 4)), dim3(256), 0, stream, X, M, K, ldx, MP, Xt, S, flags);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

int launch_rotate_rows(const _Float16* X, int64_t M, int64_t K, int64_t ldx, int mt, int groups, _Float16* Xt, _Float16* X0, uint32_t* flags,
                       hipStream_t stream) {
    const int64_t tiles = (int64_t)mt * groups * (K / kBlock);
    hipLaunchKernelGGL(rotate_rows_kernel, dim3((unsigned)tiles), dim3(512), 0, stream, X, (int)M, (int)(K / kBlock), ldx, mt, Xt, X0, flags);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

int launch_rotate_rowmajor(const _Float16* X, int64_t M, int64_t K, int64_t ldx, _Float16* Xt, uint32_t* zero_words, int n_zero, uint32_t* flags,
                           hipStream_t stream) {
    const int64_t chunks = M * (K / kBlock);
    hipLaunchKernelGGL(rotate_rowmajor_kernel, dim3((unsigned)((chunks + 15) / 16)), dim3(256), 0, stream, X, chunks, (int)(K / kBlock), ldx, Xt, zero_words, n_zero, flags);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

}  // namespace itq3s
