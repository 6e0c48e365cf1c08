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
__device__ __forceinline__ floatx4 rotate_f32(half4 xa, const half4& q) {
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    const floatx4 T = __builtin_amdgcn_mfma_f32_16x16x16f16(xa, q, zero, 0, 0, 0);
    const half4 th = __builtin_convertvector(T, half4);
    float minus_one = -1.0f;
    asm("" : "+s"(minus_one));  // (with the constant in sight the multiply-add becomes a conversion and a subtraction)
    floatx4 rest;
#pragma unroll
    for (int j = 0; j < 4; ++j) rest[j] = __builtin_fmaf((float)th[j], minus_one, T[j]);  // exact
    const half4 tl = __builtin_convertvector(rest, half4);
    floatx4 U = __builtin_amdgcn_mfma_f32_16x16x16f16(q, th, zero, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16f16(q, tl, U, 0, 0, 0);
}
__device__ __forceinline__ bool rotate_operand(half4 xa, int lane, _Float16 out[4]) {
    const half4 q = hadamard_quarter(lane);
    const floatx4 U = rotate_f32(xa, q);
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
//     e = 64 g + 16 (i>>1) + t + 8 (i&1)
// of the chunk, which is where the weight kernel's shift-and-mask unpack puts the code of the same
// element (a step is one slot of the lane's four low-plane words and the slot eight further).  Xt index = (((b*8 + t)*4 + g)*MP + m)*8 + i.   S[b*MP + m] = sum_e x~_e (rounded values),
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
    // lanes whose slots are 8 apart hold the two halves of the same words: each gives the other half of its words
    const int slot = lane & 15;
    const bool upper = (slot & 8) != 0;
    const u32x2 h = __builtin_bit_cast(u32x2, half4{r[0], r[1], r[2], r[3]});
    const uint32_t keep = upper ? h.y : h.x, got = (uint32_t)row_xor_i32<8>((int)(upper ? h.x : h.y));
    *reinterpret_cast<u32x2*>(Xt + ((((int64_t)b * 8 + (slot & 7)) * 4 + (lane >> 4)) * MP + m) * 8 + (upper ? 4 : 0)) =
        u32x2{__builtin_amdgcn_perm(keep, got, upper ? 0x05040100u : 0x01000504u), __builtin_amdgcn_perm(keep, got, upper ? 0x07060302u : 0x03020706u)};
}

// Operand order of the streaming kernel for 17 and more rows (itq3s_rows.hip): rows in groups of 16 mt, a
// group's fragments (t, mt) of a block one after another, 1 KiB each -- lane l = 16 g + r of the MFMA
// operand finds its eight halves, e = 64 g + 16 (t>>1) + 4 (t&1) + (i>>1) + 8 (i&1), at 16 l.
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

// Operand order of the block-scaled kernels (itq3s_mx_rule.h): a wavefront rotates eight rows of a block and passes the fp32
// values through LDS of its own, so that a lane holds the 32 channels (row lane % 8, quarter lane / 16, even or odd slots
// by lane / 8 % 2) that one lane of the products holds; nobody waits for another.
constexpr int kMxRowStride = 296;  // floats of a row's 256 in LDS: eight groups of 32 in 36, and 8 more (16-byte reads of 8 rows x 2 groups touch all banks)
typedef float floatx32 __attribute__((ext_vector_type(32)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void rotate_mx_kernel(const _Float16* __restrict__ X, int M, int KB, int64_t ldx,
                                                              unsigned char* __restrict__ Xm, uint32_t* __restrict__ flags) {
    __shared__ __align__(16) float lds[4][8 * kMxRowStride];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tile = (int)blockIdx.x / KB, b = (int)blockIdx.x - tile * KB;  // tile of 32 rows
    unsigned char* const out = Xm + ((int64_t)tile * KB + b) * kMxBlockBytes;
    unsigned char* const meta = out + 4 * kMxStepBytes;
    float* const rows = lds[wave];
    half4 xa[8];
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
        const int m = tile * 32 + wave * 8 + rr;
        xa[rr] = half4{(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
        if (m < M) xa[rr] = *reinterpret_cast<const half4*>(X + (int64_t)m * ldx + (int64_t)b * kBlock + 16 * (lane & 15) + 4 * (lane >> 4));
    }
    // element 64 q + 16 i + s (q = lane / 16, s = lane % 16) -> group 2 q + s % 2, place 8 i + s / 2
    const half4 q = hadamard_quarter(lane);
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
        const floatx4 U = rotate_f32(xa[rr], q);
        float* const dst = rows + rr * kMxRowStride + (2 * (lane >> 4) + (lane & 1)) * 36 + ((lane & 15) >> 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[8 * i] = U[i];
    }
    if (lane == 0) {  // E
        float* const e = reinterpret_cast<float*>(meta + 384 + wave * 32);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            *reinterpret_cast<floatx4*>(e + 4 * i) = floatx4{16.0f * (float)xa[4 * i][0], 16.0f * (float)xa[4 * i + 1][0], 16.0f * (float)xa[4 * i + 2][0], 16.0f * (float)xa[4 * i + 3][0]};
    }
    __builtin_amdgcn_wave_barrier();  // (the LDS instructions of a wavefront stay in order)
    const int r8 = lane & 7, group = lane >> 3, odd = group & 1, kg = (group >> 1) & 1, step = 2 * (group >> 2) + odd;
    const float* const src = rows + r8 * kMxRowStride + group * 36;
    floatx16 r0, r1;  // even and odd fields: the conversion's two sources
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(src + 4 * i);
        r0[2 * i] = v[0];
        r1[2 * i] = v[1];
        r0[2 * i + 1] = v[2];
        r1[2 * i + 1] = v[3];
    }
    float peak = 0.f, sum = 0.f, sum1 = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        peak = __builtin_elementwise_maximum(peak, __builtin_elementwise_maximum(__builtin_fabsf(r0[i]), __builtin_fabsf(r1[i])));
        sum += r0[i];
        sum1 += r1[i];
    }
    const bool ok = peak <= 65504.0f;
    const uint32_t bits = __builtin_bit_cast(uint32_t, peak);
    // scale 2^e with peak / 2^e in (3.75, 7.5], the largest value of the format
    uint32_t e8 = (bits >> 23) - 2u + ((bits & 0x7fffffu) > 0x700000u ? 1u : 0u);
    if (peak == 0.f || !ok) e8 = 127u;
    // Three parts leave the small values of a group an error of 1.3e-5 of its largest one (root mean square), fp16 2.1e-4 of
    // themselves: the same where the largest is 16 times the others' deviation, 24 times their median.  Where the most
    // are far below it (10 of 16 of them below 2^-5 of it), the group is fp16: activations with an offset, say,
    // rotate to one large value in a block, and the outputs whose digit there is 0 are made of the others.
    // Such outputs, offset 0 / 1 / 4 / 30 deviations: 3.4e-5, 9.8e-5, 8.2e-5, 5.2e-5 (x~ in fp16 alone 2.1e-4, 2.1e-4, 2.1e-4, 1.5e-4;
    // no group in fp16 3.4e-5, 9.8e-5, 4e-4, 2.5e-3).  Of groups of normal values one in 10^7 is.
    int small = 0;
    const float few = peak * 0.03125f;
#pragma unroll
    for (int k = 0; k < 16; k += 2) {
        small += __builtin_fabsf(r0[k]) < few ? 1 : 0;
        small += __builtin_fabsf(r1[k]) < few ? 1 : 0;
    }
    const bool wide = ok && small >= 10;
    const int at = 32 * kg + 8 * wave + r8;  // lane of the products
    unsigned char* const frag = out + step * kMxStepBytes;
    if (wide) {  // eight halves for each nibble of the lane's four words, in the place of the parts' bytes
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            half8 h;
#pragma unroll
            for (int j = 0; j < 8; ++j) {  // place 8 (j / 2) + p + 4 (j % 2)
                const int k = 4 * (j / 2) + p / 2 + 2 * (j % 2);
                h[j] = (_Float16)(p % 2 == 0 ? r0[k] : r1[k]);
            }
            const u32x4 w = __builtin_bit_cast(u32x4, h);
            if (p < 3) {
                *reinterpret_cast<u32x4*>(frag + p * kMxPartBytes + at * 16) = w;
            } else {
                *reinterpret_cast<u32x2*>(frag + 1024 + at * 8) = u32x2{w.x, w.y};
                *reinterpret_cast<u32x2*>(frag + kMxPartBytes + 1024 + at * 8) = u32x2{w.z, w.w};
                *reinterpret_cast<u32x2*>(frag + 2 * kMxPartBytes + 1024 + at * 8) = u32x2{0u, 0u};
            }
        }
    } else {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const float scale = __builtin_bit_cast(float, (e8 - (p == 0 ? 0u : p == 1 ? 4u : 9u)) << 23);
            const u32x6 packed = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(r0, r1, scale);
            const floatx32 back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(packed, scale);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                r0[k] -= back[2 * k];
                r1[k] -= back[2 * k + 1];
            }
            *reinterpret_cast<u32x4*>(frag + p * kMxPartBytes + at * 16) = u32x4{packed[0], packed[1], packed[2], packed[3]};
            *reinterpret_cast<u32x2*>(frag + p * kMxPartBytes + 1024 + at * 8) = u32x2{packed[4], packed[5]};
        }
    }
    // the sum of the parts: of the values less what remains of them (fp16 groups are multiplied with digits, not with codes)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        sum -= r0[k];
        sum1 -= r1[k];
    }
    sum += sum1;
    if (wide) sum = 0.f;
    if (!ok) sum = __builtin_nanf("");
    // -S: over the eight groups
    sum += xor_lane_f32(sum, 8);
    sum += xor_lane_f32(sum, 16);
    sum += xor_lane_f32(sum, 32);
    if (lane < 8) *reinterpret_cast<float*>(meta + 256 + (8 * wave + r8) * 4) = -sum;
    int word = (int)((wide ? 0u : ok ? e8 : 0xffu) << (8 * step));
    word |= xor_lane_i32(word, 8);
    word |= xor_lane_i32(word, 32);
    if (step == 0) *reinterpret_cast<int*>(meta + at * 4) = word;
    if (!ok && flags != nullptr) atomicOr(flags, kFlagActRange);
}

int launch_rotate_mx(const _Float16* X, int64_t M, int64_t K, int64_t ldx, unsigned char* Xm, uint32_t* flags, hipStream_t stream) {
    const int64_t tiles = (M + kMxRows - 1) / kMxRows * (K / kBlock);
    hipLaunchKernelGGL(rotate_mx_kernel, dim3((unsigned)tiles), dim3(256), 0, stream, X, (int)M, (int)(K / kBlock), ldx, Xm, flags);
    return hipGetLastError() == hipSuccess ? 0 : -6;
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

}  // namespace itq3s
