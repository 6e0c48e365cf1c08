// Streaming matmul for M <= 16 activation rows (the decode path, Sec. 5.4).  The description below is
// the kernel for M <= 4, which rotates the activations itself; the variant for 5..16 rows, which
// takes them rotated from a launch in front, is described at the kernel template.
//
//   Y[m][n] = sum_b d[n,b] * ( sum_j c[n,b,j] x~[m,b,j]  -  S[m,b]  -  z[n,b] * E[m,b] )
//
// with c = q+1 the stored code, x~ = H x the rotated activation chunk rounded to fp16 (H is
// symmetric and its own inverse, Sec. 2.3: <H v, x> = <v, H x>, so the rotation is applied to the
// activations and the packed weights are consumed as stored), S[m,b] = sum_j x~[m,b,j] over those
// rounded values (it cancels the +1 of the codes exactly) and E[m,b] = 16 x[m, 256 b], the exact
// value of the same sum before rounding (H 1 = 16 e_0): the zero-point term is formed from the
// activations themselves, so the rounding of x~ is not multiplied by z.  The packed weights are read
// exactly once -- one 16-byte + one 8-byte + one 4-byte (scale) load per lane and tile -- and nothing
// dequantized is written anywhere.
//
// Contraction: v_mfma_f32_16x16x32_f16 with the activations as the A operand (rows = m) and 16
// weight rows of a tile as the B operand (columns = n), so that every accumulator of a lane belongs
// to the lane's own weight row and needs only that row's scale.  A code c placed in bits
// 10:9 of a half is the number c * 2^-15, in bits 8:7 c * 2^-17 (fp16's subnormal numbers take part in the products
// unchanged, but the products are added up with the bits that stand in front of them missing, so not further down;
// further up, at bits 11:10, a stored 3 would count as 4), so a shift of a low-plane word by a
// multiple of four gives two half2 operands with one mask each; the factors are applied together with d.  Four-row decode is bound by this arithmetic (two of 4096x11008, M = 4: 5.5 us of
// vector instructions in a launch of 11): the two positions took a sixth off a tile's share, and the rows
// are rotated together, two by two, instead of one after another.  us, a shift a pair and row after row / now, launches
// of a graph (K x N): 11008x4096 M = 1 5.9 / 5.8, M = 4 8.5 / 7.9; 28672x8192 M = 1 19.6 / 18.9, M = 4 25.6 / 24.0; two of
// 8192x28672 M = 4 39.6 / 37.0; 5120x5120 M = 4 6.4 / 6.3; three 4096x4096 M = 1 6.1 / 6.3, M = 4 7.6 / 7.5.
//
// Work split: workgroup g (8 wavefronts) owns RT or RT-1 consecutive 16-row tiles of the launch and
// all of K; wavefront w takes blocks w, w+8, ...  A step of a wavefront is one block against the
// workgroup's row tiles: the tile loads of the next step are in flight (two register buffers) while
// the wavefront rotates the 256 activations of its current block on the matrix cores, parks them in
// its private 576 M bytes of LDS in operand order, and multiplies.  No wavefront waits for another
// before the cross-wavefront sum at the end.  Every load goes through a buffer descriptor: a row
// tile the workgroup does not have gets an empty descriptor (its loads return zeros without touching
// memory), so the step is branch-free.  The kernel needs 86 to 128 registers, which leaves room for
// two workgroups per compute unit: one workgroup's start-up and final sum overlap the other's
// streaming.
#include <hip/hip_ext.h>

#include "itq3s_dev.h"
#include <atomic>
#include <type_traits>

#include "itq3s_kernels.h"
#include "itq3s_stream.h"

namespace itq3s {

constexpr int kGemvWaves = 8;      // wavefronts per workgroup
constexpr int kGemvMaxRT = 3;      // row tiles per workgroup, at most (7 registers per tile and buffer; four would cost the second workgroup per compute unit)

static thread_local LaunchTiming g_timing;  // armed and taken on the calling thread
void set_launch_timing(hipEvent_t start, hipEvent_t stop) { g_timing.start = start; g_timing.stop = stop; }
LaunchTiming take_launch_timing() {
    const LaunchTiming t = g_timing;
    g_timing = LaunchTiming{};
    return t;
}

struct GemvArgs {
    GemvTensor t[kGemvMaxGroup];
    const _Float16* X;  // activations [M][ldx]; kRotated: x~ in operand order with MP columns (from the rotation launch)
    const float* S;     // kRotated: [2][KB][MP] sums of the rounded x~ per block and row, then 16 x[m][256 b]
    uint32_t* flags;
    int64_t ldx;
    int KB, M, y_f16;
    int nt_q, nt_r;  // row tiles per workgroup: the first nt_r workgroups own nt_q + 1, the others nt_q
};

struct TileRegs {
    u32x4 lo;
    u32x2 hi;
    uint32_t sc;
    uint32_t ss;  // (sub-block variant) the lane's two sub-scales
};

// The 256-point transform on the matrix cores.  With the chunk written as a 16 x 16 matrix
// X[a][b] = x[16a + b], the Sylvester construction gives H_256 = H_16 (x) H_16, i.e.
//     (H x)[16a' + b'] = (H_16 X H_16)[a'][b'] / 16        (H_16 with entries +-1).
// Two 16x16x16 products do it: T = X (H_16/4) (fp16 inputs, exact products, fp32 sums; the factor
// keeps |T| <= 4 max|x|), then (H_16/4) T with T split into two halves (T = T_hi + T_lo keeps 22
// bits).  The accumulator layout of the first product (lane = column
// b', four rows a per lane) is exactly the B-operand layout of the second, so nothing moves between
// lanes.  A lane holds x[16 (l%16) + 4 (l/16) + 0..3] on entry and element e = 64 (l/16) + 16 r + l%16,
// r = 0..3, of the result.
// x~ = H x for one 256-chunk of each row, rounded to fp16, in operand order: half i of step t of quarter g of row m at
// half m kXsRow + g kXsQuarter + 8 t + i.  `peak` collects the largest magnitude of a rotated value; a value (or the
// intermediate T, which then turns the result into NaN) outside the fp16 range leaves it above 65504 or NaN.
// Every workgroup rotates all of X for itself, so with two to four rows this arithmetic is a good part
// of the launch: both products take the quarter of H (their factors make up the 1/16 exactly), conversions
// go in pairs, the residue of T is one mixed-precision multiply-add, the range is one NaN-propagating
// three-way maximum per two values, and the rows go through each stage together (a row alone waits for three products
// one after another).  Element e = 64 g + 16 w + slot is half 2 w + slot / 8 of step slot % 8: lanes whose slots are 8 apart
// hold the two halves of the same words, so each gives the other half of its words and both write eight bytes.
constexpr int kXsQuarter = 72, kXsRow = 4 * kXsQuarter;  // halves; 64 and 8 more: the reads of 4 rows x 4 quarters touch all banks
struct XsLane {  // what a lane needs to write its part, computed once
    _Float16* dst;
    uint32_t sel0;  // the halves of its first word; of the second: two bytes on
};
__device__ __forceinline__ XsLane xs_lane(_Float16* xs, int lane) {
    const int g = lane >> 4, slot = lane & 15;
    return XsLane{xs + g * kXsQuarter + (slot & 7) * 8 + ((slot & 8) >> 1), (slot & 8) != 0 ? 0x05040100u : 0x01000504u};
}
template <int M0, int MN, int MP>
__device__ __forceinline__ void rotate_to_lds(const u32x2 (&raw)[MP], const half4& q, const XsLane& at, float& peak) {
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    float minus_one = -1.0f;
    asm("" : "+s"(minus_one));  // (with the constant in sight the multiply-add becomes a conversion and a subtraction)
    floatx4 T[MN], U[MN];
    half4 th[MN], tl[MN];
#pragma unroll
    for (int m = 0; m < MN; ++m) T[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4, raw[M0 + m]), q, zero, 0, 0, 0);
#pragma unroll
    for (int m = 0; m < MN; ++m) th[m] = __builtin_convertvector(T[m], half4);
#pragma unroll
    for (int m = 0; m < MN; ++m) {
        U[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(q, th[m], zero, 0, 0, 0);
        floatx4 rest;
#pragma unroll
        for (int j = 0; j < 4; ++j) rest[j] = __builtin_fmaf((float)th[m][j], minus_one, T[m][j]);  // exact
        tl[m] = __builtin_convertvector(rest, half4);
    }
#pragma unroll
    for (int m = 0; m < MN; ++m) U[m] = __builtin_amdgcn_mfma_f32_16x16x16f16(q, tl[m], U[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < MN; ++m) {
        const u32x2 h = __builtin_bit_cast(u32x2, __builtin_convertvector(U[m], half4));
        const bool upper = (at.sel0 & 0x04000000u) != 0;
        const uint32_t keep = upper ? h.y : h.x, send = upper ? h.x : h.y;
        const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x128, 0xf, 0xf, true);  // row_ror:8
        *reinterpret_cast<half4*>(at.dst + (M0 + m) * kXsRow) = __builtin_bit_cast(half4, u32x2{__builtin_amdgcn_perm(keep, got, at.sel0), __builtin_amdgcn_perm(keep, got, at.sel0 + 0x02020202u)});
        peak = __builtin_elementwise_maximum(peak, __builtin_elementwise_maximum(__builtin_fabsf(U[m][0]), __builtin_fabsf(U[m][1])));
        peak = __builtin_elementwise_maximum(peak, __builtin_elementwise_maximum(__builtin_fabsf(U[m][2]), __builtin_fabsf(U[m][3])));
    }
}

// kGrouped: the launch serves several tensors (a single-tensor launch skips the lookup and the
// fetch of the unused descriptors, which are on the way to the first load).
// NBC > 0: every wavefront has exactly NBC blocks (K = 2048 NBC): the pipeline is straight-line code, for one and two
// tiles (60 to 126 registers; three tiles would take up to 156, and the second workgroup per compute unit).
// kSub: the sub-block-scale variant of the format (Sec. 4.1: 116 bytes per block), one tensor per launch:
//   Y[m][n] = sum_b d ( sum_j s[n,b,j/32] (c-1)[n,b,j] x~[m,b,j]  -  z E[m,b] ).
// A lane's 64 codes belong to two sub-blocks (low-plane words 0,1 and 2,3), whose scales are the two
// halves of one more word per lane and tile.  The operand is the signed digit times the sub-scale:
// (c 2^-14) (16 s) - s 2^-10 = (c-1) s 2^-10, exact in fp16 for 2^-4 <= s <= 4094 (the quantizer's
// sub-scales lie below 3; smaller ones lose low bits of a contribution that is small anyway), so no
// block sum S is needed.
// kRotated (5..16 rows, MP = 8 or 16; either format): the activations arrive rotated, in operand order, from a launch
// of their own (rotating 8 or 16 rows per block inside every workgroup would cost more than the
// contraction); a wavefront loads the eight fragments and the two sums of its next block straight into
// registers right behind the arithmetic of the current one, in front of the next tile loads, so that
// the in-order load counter never makes it wait for those.
// NSG = 2 (kRotated only): the workgroup owns 2 RT row tiles; a wavefront multiplies the fragments of a
// block with the first RT tiles, then with the other RT (two pipeline steps per block), so that every
// fragment fetched -- the bulk of what a workgroup pulls through its L1 with 16 rows -- serves twice
// the weights, and its latency is met once per two steps.
template <int MP, int RT, bool kGrouped, int NBC, bool kSub = false, bool kRotated = false, int NSG = 1>
// (launch bounds: the second figure is a lower bound on wavefronts per SIMD: 4 = two workgroups per
// compute unit = at most 128 registers, which every instantiation of the general pipeline meets
// without scratch (four rows against three tiles only just: what is said to cost registers below); eight rows rotated
// here run with one workgroup per compute unit)
__global__ __launch_bounds__(kGemvWaves * 64, NBC > 0 ? 3 : (MP == 8 && !kRotated) ? 2 : 4) void gemv_kernel(const GemvArgs a) {
    static_assert(!kRotated || (NBC == 0 && MP >= 8), "rotated activations: general pipeline");
    static_assert(kRotated || MP <= 8, "in-kernel rotation: at most eight rows");
    static_assert(NSG == 1 || (NSG == 2 && kRotated), "row sub-groups: with rotated activations only");
    constexpr int RTW = RT * NSG;  // row tiles of the workgroup
    constexpr int W = kGemvWaves;
    extern __shared__ __align__(16) unsigned char smem[];
    const int KB = a.KB;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform, in an SGPR
    const int g = lane >> 4, r16 = lane & 15, mm = r16 & (MP - 1);
    const int wg = (int)blockIdx.x;
    const int nt_begin = wg * a.nt_q + (wg < a.nt_r ? wg : a.nt_r);
    const int cnt = a.nt_q + (wg < a.nt_r ? 1 : 0);
    struct SlotOut {   // where the 16 outputs of a slot go (table in LDS, read back in the epilogue)
        void* Y;
        int64_t ldy;
        int64_t n0;    // first row of the tile inside its tensor
        int64_t rows;  // rows of that tensor from n0 on that exist (<= 0: slot unused)
    };
    // LDS: per wavefront MP*512 bytes of x~ (in-kernel rotation only) | red: W*RTW*MP*16 floats | slot_out[RTW]
    constexpr size_t kXsBytes = kRotated ? 0 : (size_t)W * MP * kXsRow * 2;
    _Float16* const xs = reinterpret_cast<_Float16*>(smem) + (size_t)wave * MP * kXsRow;
    float* const red = reinterpret_cast<float*>(smem + kXsBytes);
    SlotOut* const slot_out = reinterpret_cast<SlotOut*>(smem + kXsBytes + (size_t)W * RTW * MP * 16 * 4);

    // Per slot: descriptors over the K range of the tile row in codes / scales (scalar selects; all
    // tensor entries come with the first argument fetch).
    __amdgpu_buffer_rsrc_t crs[RTW], srs[RTW], urs[kSub ? RTW : 1];
    void* so_y[RTW];  // the output table's entries: written behind the first loads, they are not needed before the end
    int64_t so_ldy[RTW], so_n0[RTW], so_rows[RTW];
    // grouped: the tensor of a slot is found from the three list positions alone, and its entry is then
    // fetched from the argument block by index (one scalar load per slot, all in flight together) --
    // selecting every field among four entries took 340 scalar instructions and nine dependent fetches
    // in front of the first weight load
    [[maybe_unused]] const auto* const kargs = (const __attribute__((address_space(4))) GemvArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    [[maybe_unused]] const int vb1 = a.t[1].v_begin, vb2 = a.t[2].v_begin, vb3 = a.t[3].v_begin;
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt) {
        const uint32_t* t_codes = a.t[0].codes;
        const uint32_t* t_scales = a.t[0].scales;
        void* t_y = a.t[0].Y;
        int64_t t_n = a.t[0].N, t_ldy = a.t[0].ldy;
        int t_begin = 0;
        if constexpr (kGrouped) {
            const int tile = nt_begin + rt;
            const int ti = (tile >= vb1 ? 1 : 0) + (tile >= vb2 ? 1 : 0) + (tile >= vb3 ? 1 : 0);  // list positions ascend; unused entries hold INT_MAX
            t_codes = kargs->t[ti].codes;
            t_scales = kargs->t[ti].scales;
            t_y = kargs->t[ti].Y;
            t_n = kargs->t[ti].N;
            t_ldy = kargs->t[ti].ldy;
            t_begin = kargs->t[ti].v_begin;
        }
        const bool have = rt < cnt;
        const int64_t local = nt_begin + rt - t_begin;
        const int64_t first = have ? local * KB : 0;
        crs[rt] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(t_codes + first * kTileWords), 0, have ? KB * 1536 : 0, kRawBuffer);
        srs[rt] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(t_scales + first * kTileRows), 0, have ? KB * 64 : 0, kRawBuffer);
        if constexpr (kSub) urs[rt] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(a.t[0].subscales + first * 64), 0, have ? KB * 256 : 0, kRawBuffer);
        so_y[rt] = t_y;
        so_ldy[rt] = t_ldy;
        so_n0[rt] = local * 16;
        so_rows[rt] = have ? t_n - local * 16 : 0;
    }
    // activations; rows beyond M have an empty descriptor and read as zeros
    __amdgpu_buffer_rsrc_t xrs[kRotated ? 1 : MP];
#pragma unroll
    for (int m = 0; m < (kRotated ? 1 : MP); ++m)
        xrs[m] = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<_Float16*>(a.X), 0, kRotated ? KB * MP * 512 : m < a.M ? (int)(((int64_t)(a.M - 1) * a.ldx + (int64_t)KB * 256) * 2) : 0, kRawBuffer);
    const __amdgpu_buffer_rsrc_t sumrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.S), 0, kRotated ? 2 * KB * MP * 4 : 0, kRawBuffer);
    const int nb = KB > wave ? (KB - wave + W - 1) / W : 0;  // blocks of this wavefront: b = wave + j*W

    constexpr uint32_t kOutside = 0x80000000u;  // an offset no descriptor here covers
    const uint32_t none = nb > 0 ? 0u : kOutside;  // a wavefront without blocks (K < 2048) loads nothing
    const uint32_t off_lo = lane * 16 + none, off_hi = lane * 8 + 1024 + none, off_sc = r16 * 4 + none, off_ss = lane * 4 + none;
    // (a row's place is in the scalar offset, which costs no register)
    const uint32_t off_x = (uint32_t)((16 * r16 + 4 * g) * 2) | none;
    // rotated activations: fragment t of the block for lane (row mm, quarter g) at ((t*4 + g)*MP + mm)*16 bytes
    const uint32_t off_xf = (uint32_t)((g * MP + mm) * 16) + none, off_sum = (uint32_t)(((4 * g) & (MP - 1)) * 4) + none;
    half8 xf[kRotated ? 8 : 1];
    floatx4 sv_r = {0.f, 0.f, 0.f, 0.f}, ev_r = {0.f, 0.f, 0.f, 0.f};
    auto issue_x = [&](int j) {  // fragments and sums of step j (kRotated)
        const int b = nb > 0 ? wave + j * W : 0;
#pragma unroll
        for (int t = 0; t < 8; ++t)
            xf[t] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(xrs[0], off_xf + (uint32_t)(t * 4 * MP * 16), b * (MP * 512), 0));
        sv_r = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(sumrs, off_sum, b * (MP * 4), 0));
        ev_r = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(sumrs, off_sum, (KB + b) * (MP * 4), 0));
    };

    floatx4 acc[RTW];
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint32_t bad = 0;
    float peak = 0.f;  // largest magnitude of the rotated activations

    struct Slot {
        TileRegs t[RT];
        u32x2 xr[kRotated ? 1 : MP];
    };
    Slot ring[2];

    // loads of step j: the wavefront's activations of block wave + j*W, then that block of every row tile
    // (of sub-group SG of the row tiles)
    auto issue_sg = [&](Slot& s, int j, auto sgc) {
        constexpr int SG = decltype(sgc)::value;
        const int b = nb > 0 ? wave + j * W : 0;
        if constexpr (!kRotated) {
#pragma unroll
            for (int m = 0; m < MP; ++m) s.xr[m] = __builtin_amdgcn_raw_buffer_load_b64(xrs[m], off_x, b * 512 + (int)(m * a.ldx * 2), 0);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            s.t[rt].lo = __builtin_amdgcn_raw_buffer_load_b128(crs[SG * RT + rt], off_lo, b * 1536, kLoadNT);
            s.t[rt].hi = __builtin_amdgcn_raw_buffer_load_b64(crs[SG * RT + rt], off_hi, b * 1536, kLoadNT);
            s.t[rt].sc = __builtin_amdgcn_raw_buffer_load_b32(srs[SG * RT + rt], off_sc, b * 64, kLoadNT);
            if constexpr (kSub) s.t[rt].ss = __builtin_amdgcn_raw_buffer_load_b32(urs[SG * RT + rt], off_ss, b * 256, kLoadNT);
        }
    };
    auto issue = [&](Slot& s, int j) { issue_sg(s, j, std::integral_constant<int, 0>{}); };

    [[maybe_unused]] const half4 hq = hadamard_quarter(lane);
    [[maybe_unused]] const XsLane xs_at = xs_lane(xs, lane);
    [[maybe_unused]] const _Float16* const xs_src = xs + mm * kXsRow + g * kXsQuarter;

    auto compute_sg = [&](const Slot& s, auto sgc) {
        constexpr int SG = decltype(sgc)::value;
        [[maybe_unused]] uint32_t first[kRotated ? 1 : MP];  // lane 0 holds x[0..3] of the chunk
        float ev[4];  // E = 16 x_0 (rows m = 4g + i of the accumulators are row m & (MP-1))
        auto sums_e = [&] {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (kRotated) {
                    ev[i] = ev_r[i];
                } else {
                    ev[i] = 16.0f * f16_bits_to_f32(first[i & (MP - 1)] & 0xffffu);
                    if constexpr (MP == 8) ev[i] = (g & 1) != 0 ? 16.0f * f16_bits_to_f32(first[4 + i] & 0xffffu) : ev[i];
                }
            }
        };
        if constexpr (!kRotated) {
            if constexpr (MP > 2) {  // (E behind the products, from scalar registers)
#pragma unroll
            for (int m = 0; m < MP; ++m) first[m] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.xr[m].x);
            }
            if constexpr (MP <= 2) {
                rotate_to_lds<0, MP>(s.xr, hq, xs_at, peak);
            } else {
                rotate_to_lds<0, 2>(s.xr, hq, xs_at, peak);
                __builtin_amdgcn_sched_barrier(0);
                rotate_to_lds<2, 2>(s.xr, hq, xs_at, peak);
                if constexpr (MP > 4) {
                    rotate_to_lds<4, 2>(s.xr, hq, xs_at, peak);
                    rotate_to_lds<6, 2>(s.xr, hq, xs_at, peak);
                }
            }
            if constexpr (MP <= 2) {
#pragma unroll
            for (int m = 0; m < MP; ++m) first[m] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.xr[m].x);
                sums_e();
            }
            // (116-byte variant, one row: without the line here the scheduler spreads the rotation over the
            // unpacking and three row tiles take 128 registers and scratch: 8192x11008 11.3 us instead of 10.7)
            if constexpr (kSub && MP == 1) __builtin_amdgcn_sched_barrier(0);
        }
        // the block sums S come from the matrix cores as well: the same fragments against an operand of ones
        uint32_t one = 0x04000400u;
        if constexpr (!kRotated && MP > 2 && RT == 3) asm("" : "+v"(one));  // (made anew for each block: registers)
        [[maybe_unused]] const half8 ones = as_half8(one, one, one, one);  // 2^-14 each
        floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
        floatx4 c[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) c[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
        half8 sub_mul[kSub ? RT : 1], sub_add[kSub ? RT : 1];  // (sub-block variant) 16 s and -s 2^-10 of the lane's two sub-blocks
        if constexpr (kSub) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const half2v s2 = __builtin_bit_cast(half2v, s.t[rt].ss);
                const half2v m = s2 * half2v{(_Float16)16.0f, (_Float16)16.0f}, n = s2 * half2v{(_Float16)(-0.0009765625f), (_Float16)(-0.0009765625f)};
                sub_mul[rt] = half8{m.x, m.x, m.x, m.x, m.y, m.y, m.y, m.y};  // words 0,1 | 2,3
                sub_add[rt] = half8{n.x, n.x, n.x, n.x, n.y, n.y, n.y, n.y};
            }
        }
        // Slots s and s + 8 of a low-plane word are 16 bits apart.  Shifted by a multiple of four the word has one pair at bits
        // 10:9 (odd s: the halves c 2^-15) and one at 8:7 (even s: c 2^-17, in a sum of its own that counts four times):
        // twelve instructions a word instead of sixteen with a shift for each pair.  (The sub-scaled operands, whose
        // range ends at fp16's, all come from bits 11:10.)
        auto fragment = [&](int t) -> half8 {
            if constexpr (kRotated) return xf[t];
            else return *reinterpret_cast<const half8*>(xs_src + 8 * t);
        };
        constexpr uint32_t kSubMask = 0x0C000C00u, kOddMask = 0x06000600u, kEvenMask = 0x01800180u;
        auto shifted = [](uint32_t v, int by) -> uint32_t { return by >= 0 ? v << by : v >> -by; };
        if constexpr (kSub) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const half8 Xf = fragment(t);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const u32x4 v = s.t[rt].lo;
                    half8 op = as_half8(shifted(v.x, 10 - 2 * t) & kSubMask, shifted(v.y, 10 - 2 * t) & kSubMask, shifted(v.z, 10 - 2 * t) & kSubMask, shifted(v.w, 10 - 2 * t) & kSubMask);
                    op = __builtin_elementwise_fma(op, sub_mul[rt], sub_add[rt]);
                    c[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Xf, op, c[rt], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            floatx4 ce[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) ce[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < 4; ++p) {  // slots 2p + 1 and 2p
                const half8 Xo = fragment(2 * p + 1), Xe = fragment(2 * p);
                if constexpr (!kRotated) {
                    sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(Xo, ones, sacc, 0, 0, 0);
                    sacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(Xe, ones, sacc, 0, 0, 0);
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const u32x4 lo = s.t[rt].lo;
                    const uint32_t v[4] = {shifted(lo.x, 7 - 4 * p), shifted(lo.y, 7 - 4 * p), shifted(lo.z, 7 - 4 * p), shifted(lo.w, 7 - 4 * p)};
                    c[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Xo, as_half8(v[0] & kOddMask, v[1] & kOddMask, v[2] & kOddMask, v[3] & kOddMask), c[rt], 0, 0, 0);
                    ce[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Xe, as_half8(v[0] & kEvenMask, v[1] & kEvenMask, v[2] & kEvenMask, v[3] & kEvenMask), ce[rt], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) c[rt][i] = __builtin_fmaf(ce[rt][i], 4.0f, c[rt][i]);
        }
        if constexpr (kRotated || MP > 2) sums_e();
        float sv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[i] = kRotated ? sv_r[i] : 16384.0f * sacc[i];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            bad |= s.t[rt].hi.x | s.t[rt].hi.y;
            const float d = f16_bits_to_f32(s.t[rt].sc & 0xffffu);
            const float z = f16_bits_to_f32(s.t[rt].sc >> 16);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[SG * RT + rt][i] = kSub       ? __builtin_fmaf(d, __builtin_fmaf(c[rt][i], 1024.0f, -z * ev[i]), acc[SG * RT + rt][i])
                                                  : __builtin_fmaf(d, __builtin_fmaf(c[rt][i], 32768.0f, -__builtin_fmaf(z, ev[i], sv[i])), acc[SG * RT + rt][i]);
        }
    };
    auto compute = [&](const Slot& s) { compute_sg(s, std::integral_constant<int, 0>{}); };

    // ---- pipeline, one step ahead; every load issued belongs to a real step (the scheduling
    // barriers keep the loads in front of the arithmetic they overlap with)
    issue(ring[0], 0);
    if constexpr (kRotated) issue_x(0);
    __builtin_amdgcn_sched_barrier(0);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int rt = 0; rt < RTW; ++rt) slot_out[rt] = SlotOut{so_y[rt], so_ldy[rt], so_n0[rt], so_rows[rt]};
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NBC > 0) {
#pragma unroll
        for (int q = 0; q < NBC; ++q) {
            if (q + 1 < NBC) issue(ring[(q + 1) & 1], q + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(ring[q & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (NSG == 2) {
        // two steps per block: ring[0] carries the first RT row tiles of a block, ring[1] the others
        constexpr std::integral_constant<int, 0> sg0{};
        constexpr std::integral_constant<int, 1> sg1{};
        int j = 0;
        for (; j + 1 < nb; ++j) {
            issue_sg(ring[1], j, sg1);
            __builtin_amdgcn_sched_barrier(0);
            compute_sg(ring[0], sg0);
            __builtin_amdgcn_sched_barrier(0);
            issue_sg(ring[0], j + 1, sg0);
            __builtin_amdgcn_sched_barrier(0);
            compute_sg(ring[1], sg1);
            __builtin_amdgcn_sched_barrier(0);
            issue_x(j + 1);
        }
        if (nb > 0) {
            issue_sg(ring[1], j, sg1);
            __builtin_amdgcn_sched_barrier(0);
            compute_sg(ring[0], sg0);
            __builtin_amdgcn_sched_barrier(0);
            compute_sg(ring[1], sg1);
        }
    } else {
        int j = 0;
        for (; j + 2 < nb; j += 2) {
            issue(ring[1], j + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(ring[0]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kRotated) issue_x(j + 1);
            issue(ring[0], j + 2);
            __builtin_amdgcn_sched_barrier(0);
            compute(ring[1]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kRotated) issue_x(j + 2);
        }
        if (j + 2 == nb) {
            issue(ring[1], j + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(ring[0]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kRotated) issue_x(j + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(ring[1]);
        } else if (j + 1 == nb) {
            compute(ring[0]);
        }
    }

    // ---- add the W partial sums of every output, store Y.  red[wave][rt][m][r]; slot_out says where
    // the 16 outputs of a slot go.  (The lane's number is counted anew: held through the pipeline it costs registers.)
    const int lane_end = MP > 2 && RT == 3 ? (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) : lane, g_end = lane_end >> 4;
#pragma unroll
    for (int rt = 0; rt < RTW; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * g_end + i < MP) red[((wave * RTW + rt) * MP + 4 * g_end + i) * 16 + (lane_end & 15)] = acc[rt][i];
    __syncthreads();
    for (int o = wave * 64 + lane_end; o < RTW * 16 * MP; o += W * 64) {
        const int rr = o % (RTW * 16), m = o / (RTW * 16);  // rr = rt*16 + r: consecutive threads, consecutive n
        const int rt = rr >> 4, r = rr & 15;
        const SlotOut so = slot_out[rt];
        if (r < so.rows && m < a.M) {
            float sum = 0.f;
#pragma unroll
            for (int wv = 0; wv < W; ++wv) sum += red[((wv * RTW + rt) * MP + m) * 16 + r];
            const int64_t n = so.n0 + r;
            if (a.y_f16) reinterpret_cast<_Float16*>(so.Y)[m * so.ldy + n] = (_Float16)sum;
            else reinterpret_cast<float*>(so.Y)[m * so.ldy + n] = sum;
        }
    }
    if (a.flags != nullptr) {
        const uint32_t f = (bad != 0u ? kFlagBadCode : 0u) | (peak <= 65504.0f ? 0u : kFlagActRange);
        if (f != 0u) atomicOr(a.flags, f);
    }
}

template <int MP, int RT, bool kGrouped, int NBC, bool kSub = false, bool kRotated = false, int NSG = 1>
static int launch_kernel(const GemvArgs& a, int grid, hipStream_t stream) {
    auto kern = gemv_kernel<MP, RT, kGrouped, NBC, kSub, kRotated, NSG>;
    const size_t lds = (kRotated ? 0 : (size_t)kGemvWaves * MP * kXsRow * 2) + (size_t)kGemvWaves * RT * NSG * MP * 16 * 4 + (size_t)RT * NSG * 32;
    const LaunchTiming tm = take_launch_timing();
    if (tm.start != nullptr) hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kGemvWaves * 64), lds, stream, tm.start, tm.stop, 0, a);
    else hipLaunchKernelGGL(kern, dim3(grid), dim3(kGemvWaves * 64), lds, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

template <int MP, int RT, int NBC>
static int launch_one(const GemvArgs& a, int grid, hipStream_t stream) {
    if (a.t[1].v_begin != 0x7fffffff) return launch_kernel<MP, RT, true, NBC>(a, grid, stream);
    return launch_kernel<MP, RT, false, NBC>(a, grid, stream);
}

template <int MP, int NBC>
static int launch_shape(const GemvArgs& a, int grid, int rt, hipStream_t stream) {
    switch (rt) {
        case 1: return launch_one<MP, 1, NBC>(a, grid, stream);
        case 2: return launch_one<MP, 2, NBC>(a, grid, stream);
        case 3: return launch_one<MP, 3, 0>(a, grid, stream);  // (straight-line code for three tiles takes more than 128 registers)
    }
    return -2;
}

template <int MP>
static int launch_blocks(const GemvArgs& a, int grid, int rt, hipStream_t stream) {
    if (a.t[0].subscales != nullptr) {  // the sub-block variant: one tensor, the general pipeline
        switch (rt) {
            case 1: return launch_kernel<MP, 1, false, 0, true>(a, grid, stream);
            case 2: return launch_kernel<MP, 2, false, 0, true>(a, grid, stream);
            case 3: return launch_kernel<MP, 3, false, 0, true>(a, grid, stream);
        }
        return -2;
    }
    if (a.KB == 8) return launch_shape<MP, 1>(a, grid, rt, stream);
    if (a.KB == 16) return launch_shape<MP, 2>(a, grid, rt, stream);
    return launch_shape<MP, 0>(a, grid, rt, stream);
}

int cu_count() {
    static std::atomic<int> n_cached{0};
    int n = n_cached.load(std::memory_order_relaxed);
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) n = v;
        else n = 256;
        n_cached.store(n, std::memory_order_relaxed);
    }
    return n;
}

int launch_gemv(const GemvWeight* w, int count, int64_t K, const _Float16* X, int64_t ldx, int64_t M, int y_f16, uint32_t* flags,
                hipStream_t stream) {
    if (count < 1 || count > kGemvMaxGroup || M < 1) return -2;
    GemvArgs a;
    a.X = X; a.S = nullptr; a.flags = flags; a.ldx = ldx; a.KB = (int)(K / kBlock); a.M = (int)M; a.y_f16 = y_f16;
    const int64_t nt_total = fill_tensors(a.t, w, count);
    if (nt_total < 0) return -2;
    // Row tiles per workgroup (every workgroup rotates all of X for itself, so more tiles per workgroup
    // mean less of that; fewer mean more workgroups in flight): as many as keep one workgroup per compute unit busy, at
    // most three; two where three would leave units with twice the tiles of others and two do not (between three
    // and four tiles a unit).  us with one / two / three tiles: three 4096x4096 M = 1 6.2 / 6.6 / 6.2, M = 4 9.2 / 8.0 / 7.0;
    // two of 4096x11008 M = 1 10.2 / 9.1 / 8.4, M = 4 14.3 / 11.3 / 10.6; 2048x16384 (four tiles a unit) M = 1 5.0 / 4.6 / 5.2, M = 4 6.9 / 5.7 / 6.3.
    const int cus = cu_count();
    int64_t want = (nt_total + cus - 1) / cus;
    if (want > kGemvMaxRT) want = nt_total <= 4 * (int64_t)cus ? 2 : kGemvMaxRT;
    int64_t grid64 = (nt_total + want - 1) / want;
    if (grid64 < cus && nt_total >= cus) grid64 = cus;  // (workgroups then own `want` or `want - 1` tiles)
    if (grid64 > 0x7fffffff) return -2;
    const int grid = (int)grid64;
    const int rt = (int)((nt_total + grid - 1) / grid);
    a.nt_q = (int)(nt_total / grid);
    a.nt_r = (int)(nt_total % grid);
    if (M > kGemvFusedMaxM) {
        if (M > kGemvSubFusedMaxM || a.t[0].subscales == nullptr) return -2;
        switch (rt) {
            case 1: return launch_kernel<8, 1, false, 0, true>(a, grid, stream);
            case 2: return launch_kernel<8, 2, false, 0, true>(a, grid, stream);
            case 3: return launch_kernel<8, 3, false, 0, true>(a, grid, stream);
        }
        return -2;
    }
    switch (M) {
        case 1: return launch_blocks<1>(a, grid, rt, stream);
        case 2: return launch_blocks<2>(a, grid, rt, stream);
        default: return launch_blocks<4>(a, grid, rt, stream);
    }
}

// Five to eight rows: rotating them in every workgroup is 128 chunks per 4096 channels, about 1 us where a
// compute unit has one workgroup, against 2.7 us for the launch in front: 4096x11008 10.5 -> 9.8 us, 4096x4096
// 6.7 -> 6.3, but 11008x4096 10.5 -> 11.7 and 28672x8192 30 -> 34.  (Both ways compute the same bits.  The
// 100-byte format keeps to the launch: its block sums come out of it rounded differently, and a
// grouped call, which may have several workgroups per unit, must equal the single ones.)
bool gemv_sub_fused(int64_t M, int64_t N, int64_t K, int64_t ldx) {
    if (M <= kGemvFusedMaxM) return true;
    return M <= kGemvSubFusedMaxM && K <= 4096 && (N + 15) / 16 <= (int64_t)kGemvMaxRT * cu_count() && (M - 1) * ldx + K <= (1LL << 29);
}

template <int MP>
static int launch_rotated(const GemvArgs& a, int grid, int rt, hipStream_t stream) {
    const bool grouped = a.t[1].v_begin != 0x7fffffff;
    if (a.t[0].subscales != nullptr) {  // the sub-block variant: one tensor per launch
        switch (rt) {
            case 1: return launch_kernel<MP, 1, false, 0, true, true>(a, grid, stream);
            case 2: return launch_kernel<MP, 2, false, 0, true, true>(a, grid, stream);
            case 3: case 4: return launch_kernel<MP, 2, false, 0, true, true, 2>(a, grid, stream);
        }
        return -2;
    }
    switch (rt) {
        case 1: return grouped ? launch_kernel<MP, 1, true, 0, false, true>(a, grid, stream) : launch_kernel<MP, 1, false, 0, false, true>(a, grid, stream);
        case 2: return grouped ? launch_kernel<MP, 2, true, 0, false, true>(a, grid, stream) : launch_kernel<MP, 2, false, 0, false, true>(a, grid, stream);
        case 3: case 4: return grouped ? launch_kernel<MP, 2, true, 0, false, true, 2>(a, grid, stream) : launch_kernel<MP, 2, false, 0, false, true, 2>(a, grid, stream);
    }
    return -2;
}

int launch_gemv_rows(const GemvWeight* w, int count, int64_t K, const _Float16* Xt, const float* S, int64_t M, int MP, int y_f16,
                     uint32_t* flags, hipStream_t stream) {
    if (count < 1 || count > kGemvMaxGroup || M <= kGemvFusedMaxM || M > kGemvMaxM || (MP != 8 && MP != 16) || M > MP) return -2;
    GemvArgs a;
    a.X = Xt; a.S = S; a.flags = flags; a.ldx = 0; a.KB = (int)(K / kBlock); a.M = (int)M; a.y_f16 = y_f16;
    const int64_t nt_total = fill_tensors(a.t, w, count);
    if (nt_total < 0) return -2;
    // Every workgroup pulls all of the rotated activations (2 MP K bytes) through its compute unit's
    // L1: as many row tiles per workgroup as keep every compute unit busy, at most four (two steps of
    // two tiles per block).
    const int cus = cu_count();
    int64_t want = (nt_total + cus - 1) / cus;
    if (want > 4) want = 4;
    int64_t grid64 = (nt_total + want - 1) / want;
    if (grid64 < cus && nt_total >= cus) grid64 = cus;
    if (grid64 > 0x7fffffff) return -2;
    const int grid = (int)grid64;
    const int rt = (int)((nt_total + grid - 1) / grid);
    a.nt_q = (int)(nt_total / grid);
    a.nt_r = (int)(nt_total % grid);
    return MP == 8 ? launch_rotated<8>(a, grid, rt, stream) : launch_rotated<16>(a, grid, rt, stream);
}

}  // namespace itq3s
