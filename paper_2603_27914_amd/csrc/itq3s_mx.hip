// Matmul for 17 and more activation rows on block-scaled matrix instructions, K shared out inside a workgroup (the sizes
// between the many-row kernel and the tiled one, which has the same arithmetic: itq3s_mx_rule.h).
//
//   Y[m][n] = sum_b d ( sum_j q[n,b,j] x~[m,b,j]  -  z E[m,b] ),   q = c - 1,  E[m,b] = 16 x[m][256 b]
//
// The codes are fp4 as they are stored: those of a low-plane word's even slots, masked (one instruction for eight
// codes), are 0, 0.5 and 1; those of its odd slots after a shift.  So no digit is ever built, where the fp16 operands
// took 13 instructions for eight weights.  The rotated activations x~ come
// in three parts of fp6 (four significant bits each) with one power of two per 32 channels of a row: x~ = 2^e (p0 + p1 / 16
// + p2 / 512), the remainder at most 2^-12 / 3.75 (6.5e-5) of the group's largest value, 3.4e-5 of the values' deviation on
// normal ones (fp16: 2.1e-4, and that is what whole products, fp32 results, are off by).  Where a group's largest value stands
// alone, the group is fp16 (rotate_mx_kernel), with products of its own (itq3s_mx_wide.h).  v_mfma_scale_f32_32x32x64_f8f6f4
// runs fp6 x fp4 at four times the fp16 rate, so three products take 0.75 of one in fp16.  The codes'
// offset (code 1 = digit 0) is taken back by starting a block's sum at -S, S the sum of its activations' parts.  A
// block's sum is a sum of its own (32 x 32 outputs in 16 registers) because its scale d belongs to a column and a
// block: one fused multiply-add per output and block.
//
// Work split: a workgroup of eight wavefronts owns 32 rows and 32 NT (KS = 8) or 64 NT (KS = 4) columns; wavefront w takes blocks
// w / (8 / KS), + KS, ... of all of K and keeps 32 x 32 NT sums; one sum over the KS wavefronts through LDS at the end, no
// other synchronisation.  Nothing is shared between wavefronts on the way: fragments and codes go straight to registers,
// a step (64 channels) ahead, codes two; the loads are spread between the products, since a wavefront that issues
// them in a row fills the address unit's queue and stands.
//
// What bounds it: no unit alone.  At 512 rows of 11008x4096 (40 us without the rotation): the way from L2 into the
// registers 62 GB/s per unit, address units 52 % and matrix pipes 33 % busy, 32 % of wavefront time waiting for loads,
// 37 % for an instruction's turn.  Measured without gain: fragments three steps ahead (NT = 3), products of one
// part side by side instead of one column's three in a row.  Whole calls, before / now, us (K x N): 4096x4096 M = 512
// 34.0 / 26.5, 11008x4096 M = 512 66 / 48, 8192x28672 M = 64 51 / 33.5, M = 24 38 / 23; 28672x8192 M = 96 83 / 50.
#include <hip/hip_ext.h>

#include <type_traits>

#include "itq3s_dev.h"
#include "itq3s_kernels.h"
#include "itq3s_mx_wide.h"
#include "itq3s_stream.h"

namespace itq3s {

struct MxTensor {
    const uint32_t* codes;
    const uint32_t* scales;
    void* Y;
    int64_t N, ldy;
    int first_item, tiles_n;  // first_item: 0x7fffffff for unused entries
};
struct MxArgs {
    MxTensor t[kGemvMaxGroup];
    const unsigned char* Xm;  // rotate_mx_kernel
    uint32_t* flags;
    int M, KB, y_f16;
    int tiles_m, items, per_chiplet, wg_per_chiplet;
};

constexpr int kMxPanel = 8;  // tiles of 32 rows

template <int KS, int NT>
__global__ __launch_bounds__(kMxWaves * 64, 2) void mx_kernel(const MxArgs args) {
    constexpr int WN = kMxWaves / KS;        // wavefronts side by side along n
    constexpr int kCols = 32 * NT * WN;      // columns of an item
    extern __shared__ __align__(16) unsigned char smem[];
    const int KB = args.KB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave / WN, wn = wave - ks * WN;  // K set and column group of the wavefront
    const int l32 = lane & 31, kg = lane >> 5;
    const int nb = KB > ks ? (KB - ks + KS - 1) / KS : 0;  // blocks of this wavefront per item: ks, ks + KS, ...

    const int item_end = min(args.items, ((int)(blockIdx.x & 7) + 1) * args.per_chiplet);
    int item = (int)(blockIdx.x & 7) * args.per_chiplet + (int)(blockIdx.x >> 3);
    if (item >= item_end) return;
    const auto* const kargs = (const __attribute__((address_space(4))) MxArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const int f1 = args.t[1].first_item, f2 = args.t[2].first_item, f3 = args.t[3].first_item;
    struct Where {
        int ti, tm, tn;
    };
    auto where = [&](int it) {
        Where w;
        w.ti = (it >= f1 ? 1 : 0) + (it >= f2 ? 1 : 0) + (it >= f3 ? 1 : 0);
        it -= kargs->t[w.ti].first_item;
        const int tiles_n = kargs->t[w.ti].tiles_n;
        const int panel = it / (kMxPanel * tiles_n), within = it - panel * (kMxPanel * tiles_n);
        const int rows = args.tiles_m - panel * kMxPanel < kMxPanel ? args.tiles_m - panel * kMxPanel : kMxPanel;
        w.tn = within / rows;
        w.tm = panel * kMxPanel + (within - w.tn * rows);
        return w;
    };
    struct Place {  // where an item's operands are, for this wavefront (no such item: empty ranges)
        __amdgpu_buffer_rsrc_t x, c, s;
    };
    auto place = [&](int it) {
        const bool have = it < item_end;
        const Where w = where(have ? it : 0);
        const int64_t nt0 = (int64_t)w.tn * (kCols / 16) + wn * (2 * NT), NTt = (kargs->t[w.ti].N + 15) >> 4;
        const int tile_rows = NTt - nt0 < 2 * NT ? (NTt > nt0 ? (int)(NTt - nt0) : 0) : 2 * NT;
        const int64_t first = tile_rows > 0 ? nt0 * KB : 0;
        Place p;
        p.x = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(args.Xm + (int64_t)w.tm * KB * kMxBlockBytes), 0, have ? KB * kMxBlockBytes : 0, kRawBuffer);
        p.c = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(kargs->t[w.ti].codes + first * kTileWords), 0, have ? tile_rows * KB * 1536 : 0, kRawBuffer);
        p.s = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(kargs->t[w.ti].scales + first * kTileRows), 0, have ? tile_rows * KB * 64 : 0, kRawBuffer);
        return p;
    };

    const int off_a = lane * 16, off_t = 1024 + lane * 8, off_m = 4 * kMxStepBytes + lane * 4;
    // codes: storage tile 2 n + l32 / 16, quarter kg of a half block, row l32 % 16; scales: that row's word
    const int off_w = (l32 >> 4) * KB * 1536 + kg * 256 + (l32 & 15) * 16, step_w = 2 * KB * 1536;
    const int off_s = (l32 >> 4) * KB * 64 + (l32 & 15) * 4, step_s = 2 * KB * 64;
    u32x4 a0[3], a1[3];  // fragments of two consecutive steps: three parts of (16 + 8) bytes a lane
    u32x2 t0[3], t1[3];
    u32x4 w0[NT], w1[NT];  // codes of two consecutive half blocks
    uint32_t sc[NT];       // scale words of the block ahead
    uint32_t mt0, mt1;
    auto issue_a = [&](u32x4 (&a)[3], u32x2 (&t)[3], const Place& p, int b, int step) {
        const int s = b * kMxBlockBytes + step * kMxStepBytes;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            a[i] = __builtin_amdgcn_raw_buffer_load_b128(p.x, off_a + i * kMxPartBytes, s, 0);
            t[i] = __builtin_amdgcn_raw_buffer_load_b64(p.x, off_t + i * kMxPartBytes, s, 0);
        }
    };
    auto issue_w = [&](u32x4 (&w)[NT], const Place& p, int b, int half) {
#pragma unroll
        for (int n = 0; n < NT; ++n) w[n] = __builtin_amdgcn_raw_buffer_load_b128(p.c, off_w + n * step_w, b * 1536 + half * 512, 0);
    };
    auto issue_m = [&](const Place& p, int b) {
        int off = off_s;
        asm volatile("" : "+v"(off));  // (the offsets are computed here and not held: registers)
#pragma unroll
        for (int n = 0; n < NT; ++n) sc[n] = __builtin_amdgcn_raw_buffer_load_b32(p.s, off + n * step_s, b * 64, 0);
        mt0 = __builtin_amdgcn_raw_buffer_load_b32(p.x, off_m, b * kMxBlockBytes, 0);
        mt1 = __builtin_amdgcn_raw_buffer_load_b32(p.x, off_m + 256, b * kMxBlockBytes, 0);
    };

    floatx16 acc[NT], blk[NT], neg_s;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    int scale_a = 0;
    float d[NT];
    const int scale_w = kDigitScales;
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    auto multiply = [&](const u32x4 (&fa)[3], const u32x2 (&ft)[3], const u32x4 (&w)[NT], auto qc) {
        constexpr int q = decltype(qc)::value;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            i32x8 op;
            if constexpr (q % 2 == 0) op = i32x8{(int)even_digits(w[n].x), (int)even_digits(w[n].y), (int)even_digits(w[n].z), (int)even_digits(w[n].w), 0, 0, 0, 0};
            else op = i32x8{(int)odd_digits(w[n].x), (int)odd_digits(w[n].y), (int)odd_digits(w[n].z), (int)odd_digits(w[n].w), 0, 0, 0, 0};
            auto part = [&](auto pc) {
                constexpr int p = decltype(pc)::value;
                const i32x8 a = {(int)fa[p].x, (int)fa[p].y, (int)fa[p].z, (int)fa[p].w, (int)ft[p].x, (int)ft[p].y, 0, 0};
                blk[n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, op, q == 0 && p == 0 ? neg_s : blk[n], 2, 4, q, scale_a, p, scale_w);
            };
            part(c0);
            part(c1);
            part(c2);
        }
    };
    uint64_t any_wide = 0;  // of the item's blocks
    float* const rowval = reinterpret_cast<float*>(smem) + wave * 64;  // -S and E of the 32 rows, this wavefront's own
    auto begin_block = [&]() {
        scale_a = (int)mt0;
        any_wide |= __builtin_amdgcn_ballot_w64(wide_steps((uint32_t)scale_a) != 0u);
        rowval[lane] = __builtin_bit_cast(float, mt1);
        __builtin_amdgcn_wave_barrier();
        uint32_t any = 0;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            d[n] = f16_bits_to_f32(sc[n] & 0xffffu);
            any |= sc[n];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const floatx4 s4 = *reinterpret_cast<const floatx4*>(rowval + 8 * i + 4 * kg);
#pragma unroll
            for (int e = 0; e < 4; ++e) neg_s[4 * i + e] = s4[e];
        }
        if (__builtin_amdgcn_ballot_w64((any & 0x7fff0000u) != 0u) != 0ull) {
            floatx4 e4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e4[i] = *reinterpret_cast<const floatx4*>(rowval + 32 + 8 * i + 4 * kg);
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const float ndz = -d[n] * f16_bits_to_f32(sc[n] >> 16);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(ndz, e4[v >> 2][v & 3], acc[n][v]);
            }
        }
    };
    auto end_block = [&]() {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(d[n], blk[n][v], acc[n][v]);
    };
    floatx4* const red = reinterpret_cast<floatx4*>(smem + kMxWaves * 256);  // [wave][4 n + i][lane]
    auto finish = [&](int it) {
        const Where w = where(it);
        const int64_t N = kargs->t[w.ti].N, ldy = kargs->t[w.ti].ldy;
        void* const Y = kargs->t[w.ti].Y;
        auto store4 = [&](const floatx4& v, int i, int64_t n) {
            const int m = w.tm * 32 + 8 * i + 4 * kg;
            if (n < N) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (m + e < args.M) {
                        if (args.y_f16) reinterpret_cast<_Float16*>(Y)[(int64_t)(m + e) * ldy + n] = (_Float16)v[e];
                        else reinterpret_cast<float*>(Y)[(int64_t)(m + e) * ldy + n] = v[e];
                    }
            }
        };
        const int64_t n0 = (int64_t)w.tn * kCols + l32;
        {
            __syncthreads();
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[(wave * (4 * NT) + 4 * n + i) * 64 + lane] = floatx4{acc[n][4 * i], acc[n][4 * i + 1], acc[n][4 * i + 2], acc[n][4 * i + 3]};
            __syncthreads();
            constexpr int kPieces = WN * NT * 4;
#pragma unroll
            for (int p0 = 0; p0 < (kPieces + kMxWaves - 1) / kMxWaves; ++p0) {
                const int p = p0 * kMxWaves + wave;
                if (p < kPieces) {
                    const int g = p / (4 * NT), rest = p - g * (4 * NT);
                    floatx4 sum = red[(g * (4 * NT) + rest) * 64 + lane];
#pragma unroll
                    for (int k = 1; k < KS; ++k) sum = sum + red[((k * WN + g) * (4 * NT) + rest) * 64 + lane];
                    store4(sum, rest & 3, n0 + (g * NT + (rest >> 2)) * 32);
                }
            }
        }
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
        if (args.flags != nullptr && w.tm == 0) {  // format check, once per tile column: the high plane must be zero
            const int64_t nt0 = (int64_t)w.tn * (kCols / 16), NTt = (N + 15) >> 4;
            const int64_t tiles = (NTt - nt0 < kCols / 16 ? NTt - nt0 : kCols / 16) * KB;
            const uint4* hp = reinterpret_cast<const uint4*>(kargs->t[w.ti].codes + nt0 * KB * kTileWords);
            uint32_t bad = 0;
#pragma unroll 4
            for (int64_t i = tid; i < tiles * 32; i += kMxWaves * 64) {
                const uint4 v = hp[(i >> 5) * (kTileWords / 4) + kTileLoWords / 4 + (i & 31)];
                bad |= v.x | v.y | v.z | v.w;
            }
            if (bad != 0u) atomicOr(args.flags, kFlagBadCode);
        }
    };

#define ITQ3S_FENCE __builtin_amdgcn_sched_barrier(0)
    // the loads between the products: issued in a row they fill the address unit's queue, and the wavefront stands
    auto spread = [&](auto qc) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(qc)::value % 2 == 0 ? 4 : 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
    };
    if (nb == 0) {  // (no block for this wavefront)
        for (; item < item_end; item += args.wg_per_chiplet) finish(item);
        return;
    }
    Place cur = place(item);
    issue_m(cur, ks);
    issue_w(w0, cur, ks, 0);
    issue_a(a0, t0, cur, ks, 0);
    int j = 0;
    while (true) {
        const bool last = j + 1 == nb;
        const int b = ks + j * KS, bn = last ? ks : b + KS;
        const Place nxt = last ? place(item + args.wg_per_chiplet) : cur;
        begin_block();
        ITQ3S_FENCE;
        issue_a(a1, t1, cur, b, 1);
        issue_w(w1, cur, b, 1);
        multiply(a0, t0, w0, c0);
        spread(c0);
        ITQ3S_FENCE;
        issue_a(a0, t0, cur, b, 2);
        multiply(a1, t1, w0, c1);
        spread(c1);
        ITQ3S_FENCE;
        issue_a(a1, t1, cur, b, 3);
        issue_w(w0, nxt, bn, 0);
        issue_m(nxt, bn);
        multiply(a0, t0, w1, c2);
        spread(c2);
        ITQ3S_FENCE;
        issue_a(a0, t0, nxt, bn, 0);
        multiply(a1, t1, w1, c3);
        spread(c3);
        ITQ3S_FENCE;
        end_block();
        ITQ3S_FENCE;
        if (last) {
            if (any_wide != 0) add_wide_steps<NT, (NT < 4 ? NT : 2)>(cur.x, cur.c, cur.s, ks, KS, nb, off_w, step_w, off_s, step_s, acc);
            any_wide = 0;
            finish(item);
            item += args.wg_per_chiplet;
            if (item >= item_end) break;
            cur = nxt;
            j = 0;
        } else {
            ++j;
        }
    }
#undef ITQ3S_FENCE
}

template <int KS, int NT>
static int launch_mx_kernel(MxArgs& a, const GemvWeight* w, int count, hipStream_t stream) {
    constexpr int kCols = 32 * NT * (kMxWaves / KS);
    constexpr int kLds = kMxWaves * 256 + kMxWaves * NT * 4096;
    int64_t items = 0;
    for (int i = 0; i < kGemvMaxGroup; ++i) {
        if (i < count) {
            a.t[i] = MxTensor{w[i].codes, w[i].scales, w[i].Y, w[i].N, w[i].ldy, (int)items, (int)((w[i].N + kCols - 1) / kCols)};
            items += (int64_t)a.tiles_m * a.t[i].tiles_n;
            if (items >= 0x7fffffff / 8) return -2;
        } else {
            a.t[i] = a.t[0];
            a.t[i].first_item = 0x7fffffff;
        }
    }
    a.items = (int)items;
    a.per_chiplet = (int)((items + 7) / 8);
    const int cus = cu_count();
    a.wg_per_chiplet = a.per_chiplet < (cus + 7) / 8 ? a.per_chiplet : (cus + 7) / 8;
    auto kern = mx_kernel<KS, NT>;
    if constexpr (kLds > 65536) {
        static DeviceOnce lds_limit;
        if (!raise_lds_limit(lds_limit, reinterpret_cast<const void*>(kern), kLds)) return -6;
    }
    const dim3 grid((unsigned)a.wg_per_chiplet * 8u), block(kMxWaves * 64);
    const LaunchTiming tm = take_launch_timing();
    if (tm.start != nullptr) hipExtLaunchKernelGGL(kern, grid, block, kLds, stream, tm.start, tm.stop, 0, a);
    else hipLaunchKernelGGL(kern, grid, block, kLds, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

int launch_mx_shares(const GemvWeight* w, int count, int64_t K, int64_t M, const unsigned char* Xm, int ks, int y_f16, uint32_t* flags, hipStream_t stream) {
    MxArgs a;
    a.Xm = Xm; a.flags = flags; a.M = (int)M; a.KB = (int)(K / kBlock); a.y_f16 = y_f16;
    a.tiles_m = (int)((M + kMxRows - 1) / kMxRows);
    if (ks == 4) return launch_mx_kernel<4, 4>(a, w, count, stream);
    int64_t N[kGemvMaxGroup];
    for (int i = 0; i < count; ++i) N[i] = w[i].N;
    switch (shares8_columns(N, count, M, K, cu_count())) {
        case 1: return launch_mx_kernel<8, 1>(a, w, count, stream);
        case 2: return launch_mx_kernel<8, 2>(a, w, count, stream);
        default: return launch_mx_kernel<8, 4>(a, w, count, stream);
    }
}

}  // namespace itq3s
