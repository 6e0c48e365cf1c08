// What the block-scaled kernels (itq3s_mx.hip, itq3s_gemm.hip) do for the steps whose activations are fp16: behind their main
// loop, which has added nothing for them (scales of 0), a pass over those steps alone, straight from memory.  So the main
// loop has neither a branch nor a register for them, and its price is a scalar OR a block (a branch in front of the products, or
// behind them, with the main loop's registers alive, put its sums into scratch).  The pass is bound by its products: four of
// 32x32x16 where a step has three at four times the rate.  us, normal activations / an offset of 4 deviations (one step of a
// block's four) / offsets of 30 that change every 64 channels (two): 4096x4096 M = 512 24.7 / 30.4 / 35.3, two 4096x11008 M = 512
// 83 / 115 / 147, two 4096x14336 M = 2048 345 / 477 / 606 (all products in fp16, a kernel for that: 34, 92, 349).
#pragma once
#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

// acc[n] += d q x~ over the wide steps of blocks first, first + stride, ... (count of them) of a tile of 32 rows (x: its
// operand) and 32 NT columns (c, s: their codes and scales; storage tile 2 n + lane % 32 / 16 at off_w + n step_w, off_s + n step_s).
// A lane's operands as in the main loop; the step's digits as halves: a code c at bits 10:9 is c 2^-15, less one.
// The next step's loads are in flight under the products of the present one.
template <int NT>
__device__ __forceinline__ void add_wide_steps(__amdgpu_buffer_rsrc_t x, __amdgpu_buffer_rsrc_t c, __amdgpu_buffer_rsrc_t s, int first, int stride, int count,
                                               int off_w, int step_w, int off_s, int step_s, floatx16 (&acc)[NT]) {
    struct Step {
        u32x4 a[4], w[NT];
        uint32_t sc[NT];
        int odd;
    };
    const int lane = lane_id();
    int base = 0;             // of 64 blocks at a time, lane i knows the i-th
    uint32_t known = 0;       // its wide steps
    uint64_t blocks = 0;      // those that have some, still to come
    uint32_t steps = 0;       // of the block at hand, still to come
    int b = 0;
    auto look = [&]() {
        const int i = base + lane;
        const uint32_t word = __builtin_amdgcn_raw_buffer_load_b32(x, i < count ? (first + i * stride) * kMxBlockBytes + 4 * kMxStepBytes : 0, 0, 0);
        known = i < count ? wide_steps(word) : 0u;
        blocks = __builtin_amdgcn_ballot_w64(known != 0u);
    };
    look();
    auto next = [&](Step& t) -> bool {
        while (steps == 0) {
            while (blocks == 0) {
                base += 64;
                if (base >= count) return false;
                look();
            }
            const int i = __builtin_ctzll(blocks);
            blocks &= blocks - 1;
            steps = (uint32_t)__builtin_amdgcn_readlane((int)known, i);
            b = first + (base + i) * stride;
        }
        const int q = __builtin_ctz(steps) >> 3;
        steps &= steps - 1;
        const int at = b * kMxBlockBytes + q * kMxStepBytes;
        int lane16 = lane * 16, lane8 = 1024 + lane * 8;
#pragma unroll
        for (int p = 0; p < 3; ++p) t.a[p] = __builtin_amdgcn_raw_buffer_load_b128(x, lane16 + p * kMxPartBytes, at, 0);
        const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(x, lane8, at, 0), hi = __builtin_amdgcn_raw_buffer_load_b64(x, lane8 + kMxPartBytes, at, 0);
        t.a[3] = u32x4{lo.x, lo.y, hi.x, hi.y};
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            t.w[n] = __builtin_amdgcn_raw_buffer_load_b128(c, off_w + n * step_w, b * (kTileWords * 4) + (q >> 1) * 512, 0);
            t.sc[n] = __builtin_amdgcn_raw_buffer_load_b32(s, off_s + n * step_s, b * (kTileRows * 4), 0);
        }
        t.odd = q & 1;
        return true;
    };
    auto multiply = [&](const Step& t) {
        const half2v minus_one = {(_Float16)(-0x1p-15f), (_Float16)(-0x1p-15f)};
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            floatx16 part;
#pragma unroll
            for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                u32x4 op;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t v = t.w[n][i] >> (2 * t.odd);
                    op[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, (p < 3 ? v << (p < 3 ? 9 - 4 * p : 0) : v >> 3) & 0x06000600u) + minus_one);
                }
                part = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, t.a[p]), __builtin_bit_cast(half8, op), part, 0, 0, 0);
            }
            const float d = 32768.0f * f16_bits_to_f32(t.sc[n] & 0xffffu);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(d, part[v], acc[n][v]);
        }
    };
    Step even, odd;
    bool have = next(even);
    while (have) {
        have = next(odd);
        multiply(even);
        if (!have) break;
        have = next(even);
        multiply(odd);
    }
}

}  // namespace itq3s
