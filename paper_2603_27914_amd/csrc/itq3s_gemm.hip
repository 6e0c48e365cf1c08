// Tiled matmul for the calls with more activation rows or larger products than the streaming kernels take (the prefill
// path).  Operands and arithmetic are those of itq3s_mx.hip: codes in fp4 as they are stored, rotated activations in three
// parts of fp6 with a power of two per 32 channels, a block's sum apart because its scale belongs to a column and a block.
//
//   Y[m][n] = sum_b d ( sum_j q[n,b,j] x~[m,b,j]  -  z E[m,b] ),   q = c - 1,  E[m,b] = 16 x[m][256 b]
//
// Workgroup tile 64 (m) x 256 (n), four wavefronts 2 x 2, wavefront tile 32 x 128 = 1 x 4 v_mfma_scale_f32_32x32x64_f8f6f4
// (64 registers of sums and 64 of a block's); two workgroups share a compute unit (57 KiB of LDS, 246 registers), so
// every SIMD holds two wavefronts of different workgroups, whose barriers are not aligned.  A fragment is 18 bits a channel
// against the digits' 2, so a wavefront is wide: its 32 rows are read from LDS once for 128 columns.
//
// Every operand is copied global -> LDS by the memory pipe (buffer_load ... lds), half a block (128 channels) ahead of the
// arithmetic, two halves in turn, one barrier per half.  The copies are written as instructions that the compiler
// does not know as writes to LDS, so that it counts the LDS reads alone; what orders the two is the wait in sync().
// The loop is rotated by one step (64 channels): behind a barrier come the products of the step before, whose
// fragments are in registers, while the first fragments of the half are on their way; the digits of a step are unpacked
// behind the last products of the step before.  Zero-points are applied a block late, where the branch does not part
// the products from the reads that they hide.
//
// What bounds it: power and the instructions' turns.  Two 4096x14336 with 2048 rows: 340 us, 1.42 PFLOP/s, matrix pipes 54 % busy
// at 1.87 GHz; the same with activations of zero, where the clock stays up, 262 us (a loop of nothing but these products
// on random registers does 2.16 PFLOP/s at 1.64 GHz).  Vector instructions are 3.3 per product; without the copies
// 300 us, without two of the three parts 215, without the scaling by d 334.  Measured without gain: three halves in LDS,
// tiles of 64 x 128 (four or eight wavefronts), a second half of the workgroup on the other blocks of K.  Before
// (fp16 operands, 128 x 256), whole calls in us: two 4096x14336 M = 2048 403 -> 350, 14336x4096 M = 2048 250 -> 188,
// two 4096x11008 M = 512 106 -> 80.
#include <hip/hip_ext.h>

#include <type_traits>

#include "itq3s_dev.h"
#include "itq3s_kernels.h"
#include "itq3s_mx_wide.h"
#include "itq3s_stream.h"

namespace itq3s {

// One launch serves up to kGemvMaxGroup tensors: their tiles form one list.
struct GemmTensor {
    const uint32_t* codes;
    const uint32_t* scales;
    void* Y;
    int64_t N, ldy;
    int first_item, tiles_n;  // first_item: 0x7fffffff for unused entries
};
struct GemmArgs {
    GemmTensor t[kGemvMaxGroup];
    const unsigned char* Xm;  // rotate_mx_kernel
    uint32_t* flags;
    int M, KB, y_f16;
    int tiles_m, x_tiles, items, per_chiplet;  // tiles of 64 rows, and of 32
};

constexpr int kTileM = 64, kTileN = 256;  // of a workgroup
constexpr int kPanel = 512 / kTileM;       // tile rows per panel
constexpr int NT = 4;                      // 32-column tiles of a wavefront
constexpr int kThreads = 256;
constexpr int kHalfBytes = 2 * kMxStepBytes;                // of 32 rows, half a block
constexpr int kCodesAt = 2 * kHalfBytes;                     // in a slot, behind the fragments of both tiles of 32 rows
constexpr int kSlot = kCodesAt + kTileN / 16 * 512;           // half a block of everything: 26 KiB
constexpr int kMeta = 2 * kSlot, kScale = kMeta + 2 * 1024;  // what belongs to a block, by its parity: of the rows, of the columns
constexpr int kGemmLds = kScale + 2 * 1024;
static_assert(kHalfBytes == 9 * 1024 && kMxMetaBytes == 512, "copies of 1 KiB");
static_assert(2 * kGemmLds <= 160 * 1024 && kGemmLds <= 64 * 1024, "two workgroups per unit, no raised limit");

// Copies global -> LDS, 16 bytes a lane: lane l of copy i to lds + 1024 i + 16 l from its offset + 1024 i.  (No vector
// register is written; LDS is, which sync() orders for the compiler as well; and m0, which is reserved and so cannot be
// named as clobbered: nothing else in a kernel with these copies may use it, which a test reads from the assembly.)
template <int COUNT>
__device__ __forceinline__ void dma16(u32x4 rsrc, int voffset, int soffset, uint32_t lds) {
    static_assert(COUNT == 1 || COUNT == 4, "");
    if constexpr (COUNT == 1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voffset), "s"(rsrc), "s"(soffset));
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %1, %2, %3 offen offset:2048 lds\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:3072 lds" ::"s"(lds), "v"(voffset), "s"(rsrc), "s"(soffset));
}
__device__ __forceinline__ u32x4 descriptor(const void* p, int64_t bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, (uint32_t)bytes, 0x00027000u};
}

// (two wavefronts per SIMD: at most 256 registers)
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_kernel(const GemmArgs args) {
    extern __shared__ __align__(1024) char lds[];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    const int xcd = blockIdx.x & 7, slot_in = blockIdx.x >> 3;
    int item = xcd * args.per_chiplet + slot_in;
    if (slot_in >= args.per_chiplet || item >= args.items) return;
    const auto* const kargs = (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const int ti = (item >= args.t[1].first_item ? 1 : 0) + (item >= args.t[2].first_item ? 1 : 0) + (item >= args.t[3].first_item ? 1 : 0);
    const uint32_t* const codes = kargs->t[ti].codes;
    const uint32_t* const scales = kargs->t[ti].scales;
    const int64_t N = kargs->t[ti].N, ldy = kargs->t[ti].ldy;
    void* const Y = kargs->t[ti].Y;
    const int tiles_n = kargs->t[ti].tiles_n;
    item -= kargs->t[ti].first_item;
    int tm, tn;
    {   // a chiplet's run of the items goes panel by panel and column by column inside one: the workgroups that run
        // together there share eight slabs of activations and eight of weights in its L2
        const int panel = item / (kPanel * tiles_n), within = item - panel * (kPanel * tiles_n);
        const int rows = args.tiles_m - panel * kPanel < kPanel ? args.tiles_m - panel * kPanel : kPanel;
        tn = within / rows;
        tm = panel * kPanel + (within - tn * rows);
    }
    const int KB = args.KB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l32 = lane & 31, kg = lane >> 5;
    const int64_t n0 = (int64_t)tn * kTileN, nt0 = n0 >> 4, tensor_tiles = (N + 15) >> 4;
    const int tile_rows = (int)(tensor_tiles - nt0 < kTileN / 16 ? tensor_tiles - nt0 : kTileN / 16);

    // (an odd number of tiles of 32 rows, rows past N: the lane's own offset lies outside the range, zeros are read)
    const int x_tiles = 2 * tm + 1 < args.x_tiles ? 2 : 1;
    const u32x4 x_rsrc = descriptor(args.Xm + (int64_t)(2 * tm) * KB * kMxBlockBytes, (int64_t)x_tiles * KB * kMxBlockBytes);
    const u32x4 c_rsrc = descriptor(codes + nt0 * KB * kTileWords, (int64_t)tile_rows * KB * (kTileWords * 4));
    const u32x4 s_rsrc = descriptor(scales + nt0 * KB * kTileRows, (int64_t)tile_rows * KB * (kTileRows * 4));

    // Copies of half a block, seven a wavefront: wavefront w takes piece w % 2 (4 KiB) of tile w / 2 of 32 rows, 4 of the codes'
    // 16 storage tiles, and one of: the last KiB of tile 0, of tile 1, what belongs to the block's rows, and to its columns
    // (with both halves: the second time the same bytes).
    const int x_stride = KB * kMxBlockBytes;  // to the second tile
    const int voff_x = (wave >> 1) * x_stride + (wave & 1) * 4096 + lane * 16;
    int voff_w[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) voff_w[i] = (2 * (wave + 4 * i) + (lane >> 5)) * KB * (kTileWords * 4) + (lane & 31) * 16;
    const int voff_s = (lane >> 2) * KB * (kTileRows * 4) + (lane & 3) * 16;
    const int voff5 = wave == 3 ? voff_s : wave == 2 ? (lane >> 5) * x_stride + (lane & 31) * 16 : wave * x_stride + lane * 16;
    const u32x4 rsrc5 = wave == 3 ? s_rsrc : x_rsrc;
    const int step5 = wave == 3 ? kTileRows * 4 : kMxBlockBytes;  // a block further
    const int half5 = wave < 2 ? kHalfBytes : 0;                   // half a block further
    const int first5 = wave < 2 ? 8 * 1024 : wave == 2 ? 4 * kMxStepBytes : 0;
    auto copy_half = [&](int b, auto halfc) {  // into slot `half`
        constexpr int half = decltype(halfc)::value;
        // beyond the last block: empty ranges, nothing is fetched (zeros go to a buffer that is free)
        u32x4 rx = x_rsrc, rc = c_rsrc, r5 = rsrc5;
        rx.z = b < KB ? rx.z : 0u;
        rc.z = b < KB ? rc.z : 0u;
        r5.z = b < KB ? r5.z : 0u;
        const uint32_t dst = lds_base + (uint32_t)(half * kSlot);
        const uint32_t dst5 = wave < 2 ? dst + (uint32_t)(wave * kHalfBytes + 8 * 1024) : lds_base + (uint32_t)((wave == 2 ? kMeta : kScale) + (b & 1) * 1024);
        dma16<1>(r5, voff5, b * step5 + half * half5 + first5, dst5);
        dma16<4>(rx, voff_x, b * kMxBlockBytes + half * kHalfBytes, dst + (uint32_t)((wave >> 1) * kHalfBytes + (wave & 1) * 4096));
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16<1>(rc, voff_w[i], b * (kTileWords * 4) + half * 512, dst + (uint32_t)(kCodesAt + (wave + 4 * i) * 1024));
    };

    u32x4 a0[3], a1[3];  // fragments of two consecutive steps: three parts of (16 + 8) bytes a lane
    u32x2 t0[3], t1[3];
    u32x4 w[NT];    // codes of a half block: quarter kg of the half
    i32x8 op[NT];  // their digits: of the step that is multiplied, then of the next
    const uint32_t a_off = (uint32_t)(wm * kHalfBytes + lane * 16), t_off = (uint32_t)(wm * kHalfBytes + 1024 + lane * 8);
    const uint32_t w_off = (uint32_t)(kCodesAt + (wn * NT * 2 + (l32 >> 4)) * 512 + kg * 256 + (l32 & 15) * 16);
    auto load_a = [&](u32x4 (&a)[3], u32x2 (&t)[3], int slot, int step) {
        const char* const base = lds + slot * kSlot + step * kMxStepBytes;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            a[p] = *reinterpret_cast<const u32x4*>(base + a_off + p * kMxPartBytes);
            t[p] = *reinterpret_cast<const u32x2*>(base + t_off + p * kMxPartBytes);
        }
    };
    auto load_w = [&](int slot) {
#pragma unroll
        for (int n = 0; n < NT; ++n) w[n] = *reinterpret_cast<const u32x4*>(lds + slot * kSlot + w_off + n * 1024);
    };
    auto unpack = [&](int n, auto step) {
        if constexpr (step == 0) op[n] = i32x8{(int)even_digits(w[n].x), (int)even_digits(w[n].y), (int)even_digits(w[n].z), (int)even_digits(w[n].w), 0, 0, 0, 0};
        else op[n] = i32x8{(int)odd_digits(w[n].x), (int)odd_digits(w[n].y), (int)odd_digits(w[n].z), (int)odd_digits(w[n].w), 0, 0, 0, 0};
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
    auto product = [&](const u32x4 (&fa)[3], const u32x2 (&ft)[3], auto qc, auto pc, int n) {
        constexpr int q = decltype(qc)::value, p = decltype(pc)::value;
        const i32x8 a = {(int)fa[p].x, (int)fa[p].y, (int)fa[p].z, (int)fa[p].w, (int)ft[p].x, (int)ft[p].y, 0, 0};
        blk[n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, op[n], q == 0 && p == 0 ? neg_s : blk[n], 2, 4, q, scale_a, p, scale_w);
    };
    // a step's products; behind the last one of a column its digits for the next step
    auto all = [&](const u32x4 (&fa)[3], const u32x2 (&ft)[3], auto qc, auto next_step) {
#pragma unroll
        for (int n = 0; n < NT; ++n) product(fa, ft, qc, c0, n);
#pragma unroll
        for (int n = 0; n < NT; ++n) product(fa, ft, qc, c1, n);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            product(fa, ft, qc, c2, n);
            unpack(n, next_step);
        }
    };
    uint32_t any_wide = 0;
    auto order = [&](auto reads, auto head, auto next_step) {
        constexpr int kReads = decltype(reads)::value, kHead = decltype(head)::value, kUnpack = decltype(next_step)::value == 0 ? 4 : 8;
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if constexpr (kHead > 0) __builtin_amdgcn_sched_group_barrier(0x002, kHead, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, kUnpack, 0);
        }
    };
    constexpr std::integral_constant<int, NT + 6> first_reads{};
    constexpr std::integral_constant<int, 6> second_reads{};
    constexpr std::integral_constant<int, 16> sixteen{};

    // what belongs to a block, read at its start; returns whether it has zero-points
    const uint32_t sc_off = (uint32_t)(kScale + (wn * NT * 2 + (l32 >> 4)) * 64 + (l32 & 15) * 4);
    auto begin_block = [&](int b) -> bool {
        const char* const meta = lds + kMeta + (b & 1) * 1024 + wm * kMxMetaBytes;
        scale_a = *reinterpret_cast<const int*>(meta + lane * 4);
        uint32_t any = 0;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const uint32_t sw = *reinterpret_cast<const uint32_t*>(lds + (b & 1) * 1024 + sc_off + n * 128);
            d[n] = f16_bits_to_f32(sw & 0xffffu);
            any |= sw;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const floatx4 s4 = *reinterpret_cast<const floatx4*>(meta + 256 + i * 32 + kg * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) neg_s[4 * i + e] = s4[e];
        }
        return __builtin_amdgcn_ballot_w64((any & 0x7fff0000u) != 0u) != 0ull;
    };
    // Zero-point terms of a block that has some in this wavefront's columns (rare: one block in a thousand; a block
    // whose first channel is an outlier has them in every column).
    auto zero_points = [&](int b) {
        const char* const meta = lds + kMeta + (b & 1) * 1024 + wm * kMxMetaBytes;
        floatx4 e4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e4[i] = *reinterpret_cast<const floatx4*>(meta + 384 + i * 32 + kg * 16);
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const uint32_t sw = *reinterpret_cast<const uint32_t*>(lds + (b & 1) * 1024 + sc_off + n * 128);
            const float ndz = -f16_bits_to_f32(sw & 0xffffu) * f16_bits_to_f32(sw >> 16);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(ndz, e4[v >> 2][v & 3], acc[n][v]);
        }
    };
    // Before a half: its copies, issued a half ago, have landed, and nobody reads the half before any more.
    auto sync = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
#define ITQ3S_FENCE __builtin_amdgcn_sched_barrier(0)

    asm volatile("s_nop 4");  // (scalar registers that a vector instruction wrote are ready for the copies)
    copy_half(0, c0);
    bool have_z = false;
    for (int b = 0; b < KB; ++b) {
        // First half.  The last step of the block before is multiplied behind the barrier, while the first
        // operands of this one are on their way.
        sync();
        if (have_z) zero_points(b - 1);
        load_w(0);
        load_a(a0, t0, 0, 0);
        if (b > 0) {
            all(a1, t1, c3, c0);
        } else {
#pragma unroll
            for (int n = 0; n < NT; ++n) unpack(n, c0);
        }
        order(first_reads, c0, c0);
        ITQ3S_FENCE;
        copy_half(b, c1);
        float dl[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) dl[n] = d[n];
        have_z = begin_block(b);
        ITQ3S_FENCE;
        load_a(a1, t1, 0, 1);
        if (b > 0) {
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(dl[n], blk[n][v], acc[n][v]);
        }
        all(a0, t0, c0, c1);
        order(second_reads, sixteen, c1);
        ITQ3S_FENCE;
        // second half
        sync();
        load_w(1);
        load_a(a0, t0, 1, 0);
        all(a1, t1, c1, c0);
        order(first_reads, c0, c0);
        ITQ3S_FENCE;
        copy_half(b + 1, c0);
        ITQ3S_FENCE;
        load_a(a1, t1, 1, 1);
        any_wide |= wide_steps((uint32_t)scale_a);
        all(a0, t0, c2, c1);
        order(second_reads, c0, c1);
        ITQ3S_FENCE;
    }
    if (have_z) zero_points(KB - 1);
    all(a1, t1, c3, c0);
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = __builtin_fmaf(d[n], blk[n][v], acc[n][v]);
    if (__builtin_amdgcn_ballot_w64(any_wide != 0u) != 0 && wm < x_tiles) {  // (no second tile of 32 rows: its scales are read as 0 too)
        const int64_t tile0 = nt0 + wn * (2 * NT);
        const int rows = tensor_tiles - tile0 < 2 * NT ? (tensor_tiles > tile0 ? (int)(tensor_tiles - tile0) : 0) : 2 * NT;
        const int64_t from = rows > 0 ? tile0 * KB : 0;
        add_wide_steps<NT, NT>(
            __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(args.Xm + (int64_t)(2 * tm + wm) * KB * kMxBlockBytes), 0, wm < x_tiles ? KB * kMxBlockBytes : 0, kRawBuffer),
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(codes + from * kTileWords), 0, rows * KB * (kTileWords * 4), kRawBuffer),
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(scales + from * kTileRows), 0, rows * KB * (kTileRows * 4), kRawBuffer), 0, 1, KB,
            (l32 >> 4) * KB * (kTileWords * 4) + kg * 256 + (l32 & 15) * 16, 2 * KB * (kTileWords * 4), (l32 >> 4) * KB * (kTileRows * 4) + (l32 & 15) * 4,
            2 * KB * (kTileRows * 4), acc);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the copies beyond the last block are into this workgroup's LDS too)
#undef ITQ3S_FENCE

    if (args.flags != nullptr && tm == 0) {  // format check, once per tile column: the high plane must be zero
        const uint4* hp = reinterpret_cast<const uint4*>(codes + nt0 * KB * kTileWords);
        const int64_t tiles = (int64_t)tile_rows * KB;
        uint32_t bad = 0;
#pragma unroll 2
        for (int64_t i = tid; i < tiles * 32; i += kThreads) {
            const uint4 v = hp[(i >> 5) * (kTileWords / 4) + kTileLoWords / 4 + (i & 31)];
            bad |= v.x | v.y | v.z | v.w;
        }
        if (bad != 0u) atomicOr(args.flags, kFlagBadCode);
    }
    // register v of a 32 x 32 tile: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
    const int64_t m_first = (int64_t)tm * kTileM + wm * 32;
    const int rows = args.M - m_first < 32 ? (int)(args.M - m_first) : 32;
    auto store = [&](auto* Yt) {
        using Out = std::remove_pointer_t<decltype(Yt)>;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int64_t col = n0 + (wn * NT + n) * 32 + l32;
            Out* dst = Yt + (m_first + 4 * kg) * ldy + col;
            if (col < N) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    if (8 * (v >> 2) + 4 * kg + (v & 3) < rows) *dst = (Out)acc[n][v];
                    dst += (v & 3) == 3 ? 5 * ldy : ldy;
                }
            }
        }
    };
    if (args.y_f16) store(reinterpret_cast<_Float16*>(Y));
    else store(reinterpret_cast<float*>(Y));
}

int launch_gemm(const GemvWeight* w, int count, int64_t K, int64_t M, const unsigned char* Xm, int y_f16, uint32_t* flags, hipStream_t stream) {
    GemmArgs a;
    a.Xm = Xm; a.flags = flags; a.M = (int)M; a.KB = (int)(K / kBlock); a.y_f16 = y_f16;
    a.tiles_m = (int)((M + kTileM - 1) / kTileM);
    a.x_tiles = (int)((M + kMxRows - 1) / kMxRows);
    int64_t items = 0;
    for (int i = 0; i < kGemvMaxGroup; ++i) {
        if (i < count) {
            a.t[i] = GemmTensor{w[i].codes, w[i].scales, w[i].Y, w[i].N, w[i].ldy, (int)items, (int)((w[i].N + kTileN - 1) / kTileN)};
            items += (int64_t)a.tiles_m * a.t[i].tiles_n;
            if (items >= 0x7fffffff / 8) return -2;
        } else {
            a.t[i] = a.t[0];
            a.t[i].first_item = 0x7fffffff;
        }
    }
    a.items = (int)items;
    a.per_chiplet = (int)((items + 7) / 8);
    const dim3 grid((unsigned)a.per_chiplet * 8u), block(kThreads);
    const LaunchTiming tm = take_launch_timing();
    if (tm.start != nullptr) hipExtLaunchKernelGGL(gemm_kernel, grid, block, kGemmLds, stream, tm.start, tm.stop, 0, a);
    else hipLaunchKernelGGL(gemm_kernel, grid, block, kGemmLds, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

}  // namespace itq3s
