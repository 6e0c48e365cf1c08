// Streaming matmul for 17 and more activation rows, up to several hundred (serving batches, short prompts).
//
//   Y[m][n] = sum_k x~[m][k] * g[n][k]  -  sum_b 16 d z x[m][256 b],   g = d (c - 1)  (exact in fp16)
//
// x~ = H x is the rotated activation chunk rounded to fp16 (H is symmetric and its own inverse, Sec. 2.3),
// written in operand order by rotate_rows_kernel; 16 x[m][256 b] is the exact sum of a rotated chunk
// (H 1 = 16 e_0), so the zero-point term is formed in fp32 from the activations themselves.
//
// Work split: a workgroup of eight wavefronts owns RT consecutive 16-row tiles of the weights, 16 MT
// activation rows and all of K; wavefront w takes blocks w, w+8, ... and keeps RT x MT accumulators of
// v_mfma_f32_16x16x32_f16; one sum over the eight wavefronts through LDS at the end, no other
// synchronisation.  Because the wavefronts of a workgroup share K out among them, no fragment of x~ is
// read twice by a workgroup: fragments go straight from L2 to registers.
//
// What bounds it: the rotated activations' way into every compute unit.  A unit that computes RT tiles pulls
// in all of x~, 2 M K bytes, at the 53 bytes per clock that a unit gets from L2 into registers (130 GB/s,
// 33 TB/s over the chip, measured with a kernel that does nothing else); 11008x4096 with 64 rows: 1.4 MB
// = 10.8 us next to 3.2 us for the weights.  Behind that the unpacking (13 vector instructions per eight
// weights) and, from 48 rows on, the matrix pipes, each about the weights' time from memory.  So RT is as
// large as the registers allow -- a fragment fetched serves RT tiles -- but no larger than keeps every unit
// busy, and K is shared out inside the workgroup.
// How a launch is divided: itq3s_rows_rule.h; which calls it takes: many_row_route in itq3s_mx_rule.h (the block-scaled
// kernels fetch 2.31 bytes an activation instead of 2 and unpack in a fifth of the instructions, but start
// 2.5 us later: a longer rotation, and 32 columns where this kernel takes 16).
// Measured, whole call with the rotation launch, two passes of the kernel for 16 rows / this one, us (K x N):
// 4096x4096 M = 32 14.3 / 9.2; M = 48 10.8, three such tensors in one group 15, two of 4096x11008 23; 11008x4096 M = 48 18.9.
//
// Order of the loads: a wavefront's load counter is in order, so the weights of the next block are issued
// between the last fragments of this block that they may overtake and the first of the next: what is
// waited for inside a block has no weight load of a later block in front of it (with P = 2), and the
// weights have a whole block period to come from memory.  The pipeline runs through the ends of items.
// Measured without gain: fragments of a whole block ahead (64 rows: 4 % slower, registers), weights without
// the nontemporal hint (2..7 % slower with one group of rows, even with several).
#include <hip/hip_ext.h>

#include <type_traits>

#include "itq3s_dev.h"
#include "itq3s_kernels.h"
#include "itq3s_stream.h"

namespace itq3s {

static_assert(kRowsMinM == kGemvMaxM + 1 && kBlock == 256, "the host side counts blocks of 256");

struct RowsArgs {
    GemvTensor t[kGemvMaxGroup];
    const _Float16* Xt;  // rotated activations in operand order, see rotate_rows_kernel
    const _Float16* X0;  // first elements of the chunks, see rotate_rows_kernel
    uint32_t* flags;
    int KB, M, y_f16;
    int m_groups;            // groups of 16 MT activation rows
    int tiles;               // of all tensors
    int items, per_chiplet;  // row groups x m_groups, and a chiplet's share of them
    int wg_per_chiplet;
};

template <int MT, int RT, bool kGrouped>
__global__ __launch_bounds__(kRowsWaves * 64, 2) void rows_kernel(const RowsArgs a) {
    constexpr int W = kRowsWaves;
    constexpr int P = MT <= 2 ? 2 : 4, S = 8 / P;  // parts of a block whose fragments are fetched together, MFMA steps per part
    constexpr int kX0Stride = MT <= 2 ? 8 : 16;    // halves per (block, row quad) of X0
    extern __shared__ __align__(16) unsigned char smem[];
    const int KB = a.KB;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, r16 = lane & 15;
    const int nb = KB > wave ? (KB - wave + W - 1) / W : 0;  // blocks of this wavefront per item

    // Items: row group (RT consecutive tiles of the launch's list) x group of activation rows.  Chiplet x
    // (workgroups are dealt to the eight chiplets round-robin) takes a contiguous run of the items; the
    // row groups' m_groups are neighbours in it and share the weights in that chiplet's L2.
    const int item_end = min(a.items, ((int)(blockIdx.x & 7) + 1) * a.per_chiplet);
    int item = (int)(blockIdx.x & 7) * a.per_chiplet + (int)(blockIdx.x >> 3);
    if (item >= item_end) return;
    const auto* const kargs = (const __attribute__((address_space(4))) RowsArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const int vb1 = a.t[1].v_begin, vb2 = a.t[2].v_begin, vb3 = a.t[3].v_begin;
    struct Place {  // where an item's operands are
        __amdgpu_buffer_rsrc_t c[RT], s[RT], x, e;
    };
    // tile of the launch's list -> its tensor (list positions ascend, unused entries hold INT_MAX)
    auto tensor_of = [&](int tile) { return kGrouped ? (tile >= vb1 ? 1 : 0) + (tile >= vb2 ? 1 : 0) + (tile >= vb3 ? 1 : 0) : 0; };
    auto place = [&](int it) {
        const bool have = it < item_end;  // (no such item: empty descriptors, loads return zeros without touching memory)
        int rg = have ? it : 0, mg = 0;
        if (a.m_groups > 1) {  // (an integer division: 30 scalar instructions in front of the first load)
            const int i = rg;
            rg = i / a.m_groups;
            mg = i - rg * a.m_groups;
        }
        Place p;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int tile = rg * RT + rt, ti = tensor_of(tile);
            const bool have_t = have && tile < a.tiles;
            const int64_t at = have_t ? (int64_t)(tile - kargs->t[ti].v_begin) * KB : 0;
            p.c[rt] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(kargs->t[ti].codes + at * kTileWords), 0, have_t ? KB * 1536 : 0, kRawBuffer);
            p.s[rt] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(kargs->t[ti].scales + at * kTileRows), 0, have_t ? KB * 64 : 0, kRawBuffer);
        }
        p.x = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(a.Xt + (int64_t)mg * KB * (MT * 4096)), 0, have ? KB * (MT * 8192) : 0, kRawBuffer);
        p.e = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(a.X0 + (int64_t)mg * KB * (4 * kX0Stride)), 0, have ? KB * (8 * kX0Stride) : 0, kRawBuffer);
        return p;
    };

    const int off16 = lane * 16, off_hi = lane * 8 + 1024, off_sc = r16 * 4, off_e = g * (kX0Stride * 2);
    struct Tiles {
        u32x4 lo[RT];
        u32x2 hi[RT];
        uint32_t sc[RT];
    };
    Tiles w0, w1;
    half8 xa[S][MT], xb[S][MT];  // fragments of two consecutive parts
    u32x4 x0[kX0Stride / 8];     // first elements of a block's chunks: rows 16 mt + 4 g + i at half 4 mt + i

    auto issue_w = [&](Tiles& s, const Place& p, int b) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            s.lo[rt] = __builtin_amdgcn_raw_buffer_load_b128(p.c[rt], off16, b * 1536, kLoadNT);
            s.hi[rt] = __builtin_amdgcn_raw_buffer_load_b64(p.c[rt], off_hi, b * 1536, kLoadNT);
            s.sc[rt] = __builtin_amdgcn_raw_buffer_load_b32(p.s[rt], off_sc, b * 64, kLoadNT);
        }
    };
    // the fragments of one step of a part (and, with a block's first step, its first elements)
    auto issue_x_step = [&](half8 (&x)[S][MT], const Place& p, int b, auto partc, int t) {
        constexpr int part = decltype(partc)::value;
        if (part == 0 && t == 0) {
#pragma unroll
            for (int q = 0; q < kX0Stride / 8; ++q) x0[q] = __builtin_amdgcn_raw_buffer_load_b128(p.e, off_e + 16 * q, b * (kX0Stride * 8), 0);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int f = (S * part + t) * MT + mt;  // fragment of the block: 1 KiB each
            x[t][mt] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(p.x, off16 + (f & 3) * 1024, b * (MT * 8192) + (f >> 2) * 4096, 0));
        }
    };
    auto issue_x = [&](half8 (&x)[S][MT], const Place& p, int b, auto partc) {
#pragma unroll
        for (int t = 0; t < S; ++t) issue_x_step(x, p, b, partc, t);
    };

    floatx4 acc[RT][MT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[rt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint32_t bad = 0;

    // Eight codes of a lane (pairs p: slots p and p + 8 of a low-plane word, at bits 2p+1:2p of either half)
    // -> d (c - 1).  OR-ed into the mantissa of the half 2^(10-2p), whose bit 2p weighs exactly 1, they form
    // 2^(10-2p) + c; adding -(2^(10-2p) + 1) gives the digit exactly, times d (exact).
    auto unpack = [&](uint32_t v, half2v dd) -> half8 {
        uint32_t o[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            constexpr uint32_t kMagic[4] = {0x64006400u, 0x5C005C00u, 0x54005400u, 0x4C004C00u};  // 1024, 256, 64, 16
            constexpr float kBase[4] = {1024.0f, 256.0f, 64.0f, 16.0f};
            uint32_t bits;
            asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(bits) : "v"(v), "s"(0x00030003u << (2 * p)), "v"(kMagic[p]));
            const _Float16 o1 = (_Float16)(-(kBase[p] + 1.0f));
            o[p] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(half2v, bits) + half2v{o1, o1}) * dd);
        }
        return as_half8(o[0], o[1], o[2], o[3]);
    };
    // Zero-point terms of a block (an fp32 product per column, one fused multiply-add per output) and the
    // operands of its first step.
    half8 op[RT];
    half2v dd[RT];
    auto begin = [&](const Tiles& s) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            bad |= s.hi[rt].x | s.hi[rt].y;
            const _Float16 d = __builtin_bit_cast(_Float16, (uint16_t)(s.sc[rt] & 0xffffu));
            dd[rt] = half2v{d, d};
            const float ndz = (float)d * (-16.0f * f16_bits_to_f32(s.sc[rt] >> 16));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const half8 e8 = __builtin_bit_cast(half8, x0[mt >> 1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[rt][mt][i] = __builtin_fmaf(ndz, (float)e8[4 * (mt & 1) + i], acc[rt][mt][i]);
            }
            op[rt] = unpack(s.lo[rt].x, dd[rt]);
        }
    };
    // One part of a block.  The products of a step are issued between the unpack instructions of the next
    // step's operands.
    auto compute = [&](const Tiles& s, const half8 (&x)[S][MT], auto partc, auto&& loads) {
        constexpr int part = decltype(partc)::value;
#pragma unroll
        for (int t = 0; t < S; ++t) {
            const int next = S * part + t + 1;  // step of the block whose operands are unpacked here
            loads(t);
            half8 nop[RT];
            if (next < 8) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint32_t word = next < 2 ? s.lo[rt].x : next < 4 ? s.lo[rt].y : next < 6 ? s.lo[rt].z : s.lo[rt].w;
                    nop[rt] = unpack((next & 1) == 0 ? word : word >> 8, dd[rt]);
                }
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[rt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[t][mt], op[rt], acc[rt][mt], 0, 0, 0);
            if (next < 8) {
                constexpr int kPerProduct = (13 + MT - 1) / MT;  // 13 unpack instructions per row tile and step
#pragma unroll
                for (int r = 0; r < RT * MT; ++r) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, kPerProduct, 0);
                    if (r % RT == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) op[rt] = nop[rt];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> p0{};
    constexpr std::integral_constant<int, 1> p1{};
    constexpr std::integral_constant<int, 2> p2{};
    constexpr std::integral_constant<int, 3> p3{};

    // The sum over the eight wavefronts of an item's outputs, and their store.  red[wave][rt][mt][lane] of
    // four floats: rows 16 mt + 4 g + 0..3 of column r16.
    floatx4* const red = reinterpret_cast<floatx4*>(smem);
    auto finish = [&](int it) {
        __syncthreads();  // the previous item's sums have been read
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                red[((wave * RT + rt) * MT + mt) * 64 + lane] = acc[rt][mt];
                acc[rt][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        __syncthreads();
        const int rg = it / a.m_groups, mg = it - rg * a.m_groups;
        for (int p = wave; p < RT * MT; p += W) {
            const int rt = p / MT, mt = p - rt * MT;
            const int tile = rg * RT + rt, ti = tensor_of(tile);
            if (tile >= a.tiles) break;
            const int64_t n = (int64_t)(tile - kargs->t[ti].v_begin) * 16 + r16, ldy = kargs->t[ti].ldy, N = kargs->t[ti].N;
            void* const Y = kargs->t[ti].Y;
            const int m = (mg * MT + mt) * 16 + 4 * g;
            floatx4 sum = red[p * 64 + lane];
#pragma unroll
            for (int wv = 1; wv < W; ++wv) sum = sum + red[(wv * RT * MT + p) * 64 + lane];
            if (n < N) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (m + i < a.M) {
                        if (a.y_f16) reinterpret_cast<_Float16*>(Y)[(m + i) * ldy + n] = (_Float16)sum[i];
                        else reinterpret_cast<float*>(Y)[(m + i) * ldy + n] = sum[i];
                    }
            }
        }
    };

    // ---- one pipeline over the blocks of all items of the workgroup: while a block is multiplied, the
    // weights of the next one -- of the next item behind the last -- are on their way (the scheduling
    // barriers keep the loads in front of the arithmetic they overlap with)
#define ITQ3S_FENCE __builtin_amdgcn_sched_barrier(0)
    if (nb == 0) {  // (K < 2048: no block for this wavefront)
        for (; item < item_end; item += a.wg_per_chiplet) finish(item);
    } else {
        Place cur = place(item);
        int j = 0;
        issue_w(w0, cur, wave);
        issue_x(xa, cur, wave, p0);
        auto block = [&](const Tiles& w, Tiles& wn) -> bool {  // returns true behind the workgroup's last block
            const bool last = j + 1 == nb;
            const Place nxt = last ? place(item + a.wg_per_chiplet) : cur;
            const int b = wave + j * W, bn = last ? wave : b + W;
            issue_x(xb, cur, b, p1);
            issue_w(wn, nxt, bn);
            ITQ3S_FENCE;
            begin(w);
            ITQ3S_FENCE;
            compute(w, xa, p0, [](int) {});
            ITQ3S_FENCE;
            if constexpr (P == 2) {
                compute(w, xb, p1, [&](int t) { issue_x_step(xa, nxt, bn, p0, t); });
            } else {
                compute(w, xb, p1, [&](int t) { issue_x_step(xa, cur, b, p2, t); });
                ITQ3S_FENCE;
                compute(w, xa, p2, [&](int t) { issue_x_step(xb, cur, b, p3, t); });
                ITQ3S_FENCE;
                compute(w, xb, p3, [&](int t) { issue_x_step(xa, nxt, bn, p0, t); });
            }
            ITQ3S_FENCE;
            cur = nxt;
            if (!last) {
                ++j;
                return false;
            }
            finish(item);
            item += a.wg_per_chiplet;
            j = 0;
            return item >= item_end;
        };
        while (true) {
            if (block(w0, w1)) break;
            if (block(w1, w0)) break;
        }
    }
#undef ITQ3S_FENCE
    if (a.flags != nullptr && bad != 0u) atomicOr(a.flags, kFlagBadCode);
}

template <int MT, int RT, bool kGrouped>
static int launch_rows_kernel(const RowsArgs& a, hipStream_t stream) {
    auto kern = rows_kernel<MT, RT, kGrouped>;
    constexpr int kLds = kRowsWaves * RT * MT * 1024;
    if constexpr (kLds > 65536) {
        static DeviceOnce lds_limit;
        if (!raise_lds_limit(lds_limit, reinterpret_cast<const void*>(kern), kLds)) return -6;
    }
    const LaunchTiming tm = take_launch_timing();
    const dim3 grid((unsigned)a.wg_per_chiplet * 8u), block(kRowsWaves * 64);
    if (tm.start != nullptr) hipExtLaunchKernelGGL(kern, grid, block, kLds, stream, tm.start, tm.stop, 0, a);
    else hipLaunchKernelGGL(kern, grid, block, kLds, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

template <int MT, int RT>
static int launch_rows_rt(const RowsArgs& a, hipStream_t stream) {
    if (a.t[1].v_begin != 0x7fffffff) return launch_rows_kernel<MT, RT, true>(a, stream);
    return launch_rows_kernel<MT, RT, false>(a, stream);
}

template <int MT>
static int launch_rows_mt(const RowsArgs& a, int rt, hipStream_t stream) {
    switch (rt) {
        case 1: return launch_rows_rt<MT, 1>(a, stream);
        case 2: return launch_rows_rt<MT, 2>(a, stream);
        case 3: return launch_rows_rt<MT, 3>(a, stream);
        case 4: return launch_rows_rt<MT, 4>(a, stream);
    }
    return -2;
}

int launch_rows(const GemvWeight* w, int count, int64_t K, const _Float16* X, int64_t ldx, int64_t M, _Float16* Xt, _Float16* X0, int y_f16,
                uint32_t* flags, hipStream_t stream) {
    if (count < 1 || count > kGemvMaxGroup || M < 1 || M > kRowsMaxM || K > kRowsMaxK) return -2;
    RowsArgs a;
    a.Xt = Xt; a.X0 = X0; a.flags = flags; a.KB = (int)(K / kBlock); a.M = (int)M; a.y_f16 = y_f16;
    const int64_t nt_total = fill_tensors(a.t, w, count);
    if (nt_total < 0) return -2;
    const int cus = cu_count();
    const RowsSplit split = rows_split(nt_total, M, K, cus);
    const int mt = split.mt, rt = split.rt;
    const int groups = (int)((M + 16 * mt - 1) / (16 * mt));
    a.m_groups = groups;
    const int64_t row_groups = (nt_total + rt - 1) / rt;
    if (row_groups * groups > 0x7fffffff / 8) return -2;
    a.tiles = (int)nt_total;
    a.items = (int)(row_groups * groups);
    a.per_chiplet = (a.items + 7) / 8;
    a.wg_per_chiplet = a.per_chiplet < (cus + 7) / 8 ? a.per_chiplet : (cus + 7) / 8;
    const int rc = launch_rotate_rows(X, M, K, ldx, mt, groups, Xt, X0, flags, stream);
    if (rc != 0) return rc;
    switch (mt) {
        case 1: return launch_rows_mt<1>(a, rt, stream);
        case 2: return launch_rows_mt<2>(a, rt, stream);
        case 3: return launch_rows_mt<3>(a, rt, stream);
        case 4: return launch_rows_mt<4>(a, rt, stream);
    }
    return -2;
}

}  // namespace itq3s
