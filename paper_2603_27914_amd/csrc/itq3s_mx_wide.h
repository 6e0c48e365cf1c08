// What the block-scaled kernels (itq3s_mx.hip, itq3s_gemm.hip) do for groups of activations that are fp16: behind their main
// loop, which has added nothing for them (scales of 0), a pass over the steps that have some, straight from memory.  So the
// main loop has neither a branch nor the registers for them, and its price is three instructions a block (a branch in front of the
// products, or behind them, with the main loop's registers alive, put its sums into scratch).
// The pass is bound by its loads, 8 KB a step and wavefront through the address units, besides the products, four of 32x32x16 where a
// step has three at four times the rate.  Neither two products a group instead of four a step (two 4096x14336 M = 2048 with an
// offset 470 us, with more groups 775) nor half of the vector instructions (codes, and their offset from products with ones:
// 483 and 626) was clearly faster.
// us, normal activations / an offset of 4 deviations (one step of a block's four) / offsets of 30 that change every 64 channels (two):
// 4096x4096 M = 512 24.9 / 30.5 / 35.6, two 4096x11008 M = 512 82 / 116 / 146, two 4096x14336 M = 2048 345 / 483 / 613 (a
// kernel with fp16 operands throughout: 33, 92, 349).
#pragma once
#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

// acc[n] += d q x~ over the fp16 groups of blocks first, first + stride, ... (count of them) of a tile of 32 rows (x: its
// operand) and 32 NT columns (c, s: their codes and scales; storage tile 2 n + lane % 32 / 16 at off_w + n step_w, off_s + n step_s).
// A lane's operands as in the main loop; the step's digits as halves: a code c at bits 10:9 is c 2^-15, less one.
// The next step's loads are in flight under the products of the present one.
// (AHEAD: of the codes that many operands: mx_kernel with four holds the next item's loads besides)
template <int NT, int AHEAD>
__device__ __forceinline__ void add_wide_steps(__amdgpu_buffer_rsrc_t x, __amdgpu_buffer_rsrc_t c, __amdgpu_buffer_rsrc_t s, int first, int stride, int count,
                                               int off_w, int step_w, int off_s, int step_s, floatx16 (&acc)[NT]) {
    struct Step {
        u32x4 a[4], w[AHEAD];
        uint32_t sc[NT];
        int codes, odd;
        uint32_t mine;  // whether the lane's group is fp16 (the others' bytes are fp6)
    };
    const int lane = lane_id();
    auto look = [&](int i) {  // the lane's scales of the i-th block
        return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(x, 4 * kMxStepBytes + lane * 4, (i < count ? first + i * stride : first) * kMxBlockBytes, 0);
    };
    int i = 0, b = first;
    uint32_t wide = wide_steps(look(0)), ahead = look(1);  // of block i and the next; steps: those of any lane that are still to come
    auto of_any_lane = [&]() {
        uint32_t steps = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) steps |= __builtin_amdgcn_ballot_w64(((wide >> (8 * q + 7)) & 1u) != 0) != 0 ? 1u << q : 0u;
        return steps;
    };
    uint32_t steps = of_any_lane();
    auto next = [&](Step& t) -> bool {
        while (steps == 0) {
            if (++i >= count) return false;
            b = first + i * stride;
            wide = wide_steps(ahead);
            ahead = look(i + 1);
            steps = of_any_lane();
        }
        const int q = __builtin_ctz(steps);
        steps &= steps - 1;
        const int at = b * kMxBlockBytes + q * kMxStepBytes;
        const int lane16 = lane * 16, lane8 = 1024 + lane * 8;
#pragma unroll
        for (int p = 0; p < 3; ++p) t.a[p] = __builtin_amdgcn_raw_buffer_load_b128(x, lane16 + p * kMxPartBytes, at, 0);
        const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(x, lane8, at, 0), hi = __builtin_amdgcn_raw_buffer_load_b64(x, lane8 + kMxPartBytes, at, 0);
        t.a[3] = u32x4{lo.x, lo.y, hi.x, hi.y};
        t.codes = b * (kTileWords * 4) + (q >> 1) * 512;
#pragma unroll
        for (int n = 0; n < AHEAD; ++n) t.w[n] = __builtin_amdgcn_raw_buffer_load_b128(c, off_w + n * step_w, t.codes, 0);
#pragma unroll
        for (int n = 0; n < NT; ++n) t.sc[n] = __builtin_amdgcn_raw_buffer_load_b32(s, off_s + n * step_s, b * (kTileRows * 4), 0);
        t.odd = q & 1;
        t.mine = ((wide >> (8 * q + 7)) & 1u) != 0 ? ~0u : 0u;
        return true;
    };
    auto multiply = [&](Step& t) {
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
                    const uint32_t v = t.w[n % AHEAD][i] >> (2 * t.odd);
                    op[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, (p < 3 ? v << (p < 3 ? 9 - 4 * p : 0) : v >> 3) & 0x06000600u) + minus_one);
                }
                part = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, t.a[p] & t.mine), __builtin_bit_cast(half8, op), part, 0, 0, 0);
            }
            if (n + AHEAD < NT) t.w[n % AHEAD] = __builtin_amdgcn_raw_buffer_load_b128(c, off_w + (n + AHEAD) * step_w, t.codes, 0);
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
