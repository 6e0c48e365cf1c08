// Tiled matmul for the calls with more activation rows or larger products than the streaming kernels take
// (the prefill path): a dense contraction on the matrix cores.  Alg. 2 dequantizes a weight tile into on-chip memory and multiplies from there; here the
// operand fed to the matrix cores holds the un-rotated grid values d (q - z) in fp16 (exact for
// z = 0), the rotation having been moved to the activations (Sec. 2.3: <H v, x> = <v, H x>), so the
// weight path needs three packed-fp16 operations per pair of weights and no butterflies.
//
//   Y[m][n] = sum_k x~[m][k'] * g[n][k']  -  sum_b d z 16 x[m][256 b],   g = d (c - 1)  (exact in fp16)
//
// The zero-point multiplies the sum of the rotated chunk, and H 1 = 16 e_0 makes that sum exactly
// 16 times the chunk's first element: the term is formed from the activations themselves in fp32.
// Folding z into the fp16 operand instead would multiply the rounding errors of x~ by z.  The term
// is rare (a fraction of a percent of the blocks on real weights), so the kernel notes while it runs
// whether a zero-point came by and only then walks the scale words of its columns at the end; the
// terms are subtracted from the accumulators, so an output element is rounded once.
//
// k' is the channel order the unpack produces (within each group of 16 channels: 0,8,1,9,...,7,15);
// the rotation kernel writes x~ in the same order.  A operand = x~ rows, B operand = weight rows, so
// a lane's accumulator column is an output channel n and stores are contiguous along n.
#include <hip/hip_ext.h>

#include <type_traits>

#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

constexpr int64_t kGemmMaxK = 1 << 22;  // per-lane byte offsets (up to 128 rows x K x 2) are 32-bit

struct GemmArgs {
    const uint32_t* codes;
    const uint32_t* scales;
    const _Float16* Xt;  // [M][K] in k' order
    const _Float16* X;   // [M][ldx] the activations themselves (zero-point term)
    void* Y;
    uint32_t* flags;
    int64_t N, K, M, ldy, ldx;
    int NT, KB, y_f16;
    // split-K (splits > 1): the contraction kernel writes partial tiles [tile][split][32][256 threads]
    // of four floats and ORs 1 into zflags[tile] if it met a zero-point; a second launch adds them up
    float* partial;
    uint32_t* zflags;
    int splits;
};

// One launch serves up to kGemvMaxGroup tensors that do not split K: their tiles form one list.  Two
// tensors of 172 tiles each (11008 columns, 512 rows) leave a third of the compute units without work and
// the others with one workgroup instead of two when each has a launch of its own.
struct GemmTensor {
    const uint32_t* codes;
    const uint32_t* scales;
    void* Y;
    int64_t N, ldy;
    int first_item, tiles_n;  // first_item: 0x7fffffff for unused entries
};
struct GemmGroup {
    GemmArgs common;  // codes, scales, Y, N, ldy and NT are the tensor's
    GemmTensor t[kGemvMaxGroup];
};

// LDS accesses by raw byte address, hidden from the compiler like every other LDS read of this file
// (it would order visible LDS accesses after all outstanding global -> LDS copies).
__device__ __forceinline__ void lds_write_b32(uint32_t addr, uint32_t v) { asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_add_f32(uint32_t addr, float v) { asm volatile("ds_add_f32 %0, %1" ::"v"(addr), "v"(v) : "memory"); }

// Zero-point terms of 32 rows (m_first ..) of a wavefront's 64 columns (n_first ..), summed in fp32 in the
// accumulators' layout -- they are subtracted from the accumulators BEFORE the output is rounded: with
// fp16 outputs, correcting the stored value instead would round a sum that still contains the +z offset of
// every code and lose up to 2^-11 of that larger number.  Lane l walks the scale words of column
// n_first + l, eight blocks per batch (independent loads).  For each block in which a column has z != 0 the
// lanes exchange their columns' d z (lane -> accumulator column) and add d z 16 x[m][256 b], the 32 row
// values through 128 bytes of LDS at `xbuf` (the wavefront's own): about 60 instructions a block however many
// of its columns are concerned.  (An outlier channel at the start of a block gives every column a
// zero-point there.  Adding one column at a time to a table in LDS, as the first version did, made a launch
// of two 11008x4096 tensors with 512 rows take 174 us on such weights instead of 107.)  Per element
// the blocks are added in ascending order, so the result does not depend on scheduling.
__device__ __forceinline__ void zero_point_terms(const GemmArgs& a, int64_t n_first, int64_t m_first, int lane, uint32_t xbuf, floatx16 (&terms)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) terms[j][v] = 0.f;
    const int64_t n = n_first + lane;
    const int64_t nc = n < a.N ? n : a.N - 1;
    const uint32_t* sc = a.scales + (nc >> 4) * a.KB * kTileRows + (nc & 15);
    const bool row_ok = lane < 32 && m_first + lane < a.M;
    const _Float16* const xrow = a.X + (row_ok ? m_first + lane : 0) * a.ldx;
    const uint32_t xread = xbuf + (uint32_t)((lane >> 5) * 16);  // rows 8 q + 4 (lane / 32) + 0..3
#pragma unroll 1
    for (int b0 = 0; b0 < a.KB; b0 += 8) {
        uint32_t w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) w[u] = sc[(int64_t)(b0 + u < a.KB ? b0 + u : a.KB - 1) * kTileRows];
        uint32_t any = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (n >= a.N || b0 + u >= a.KB) w[u] = 0u;
            any |= w[u] & 0x7fff0000u;
        }
        if (__builtin_amdgcn_ballot_w64(any != 0u) == 0ull) continue;  // uniform
        _Float16 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = xrow[(int64_t)(b0 + u < a.KB ? b0 + u : a.KB - 1) * kBlock];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (__builtin_amdgcn_ballot_w64((w[u] & 0x7fff0000u) != 0u) == 0ull) continue;  // uniform
            if (lane < 32) lds_write_b32(xbuf + (uint32_t)(4 * lane), __builtin_bit_cast(uint32_t, row_ok ? 16.0f * (float)x[u] : 0.0f));
            const float dz = f16_bits_to_f32(w[u] & 0xffffu) * f16_bits_to_f32(w[u] >> 16);
            float dzc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                dzc[j] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * (32 * j + (lane & 31)), __builtin_bit_cast(int, dz)));
            floatx4 xr[4];
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:32\n\tds_read_b128 %2, %4 offset:64\n\tds_read_b128 %3, %4 offset:96\n\t"
                         "s_waitcnt lgkmcnt(0)" : "=&v"(xr[0]), "=&v"(xr[1]), "=&v"(xr[2]), "=&v"(xr[3]) : "v"(xread) : "memory");
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) terms[j][v] = __builtin_fmaf(dzc[j], xr[v >> 2][v & 3], terms[j][v]);
        }
    }
}

// The common case -- the zero-points of a wavefront's 64 columns sit in at most eight of them -- needs
// one scan for all 128 rows instead of four: one 128-row strip of floats per such column (strip_offset())
// fits the wavefront's own corner of the weight ring (1 KiB of each of its four stages: two strips
// each), so nothing is shared, nobody is waited for, and one scan serves all 128 rows.  cols receives
// the columns (0..63, -1: slot unused).  Returns false, with the strips in an undefined state, if a
// ninth column turns up.
constexpr int kStrips = 8;
struct StripColumns {
    int c[kStrips];
};
__device__ __forceinline__ uint32_t strip_offset(int slot) { return (uint32_t)((slot >> 1) * 4096 + (slot & 1) * 512); }
__device__ __forceinline__ bool zero_point_terms_few_columns(const GemmArgs& a, int64_t n_first, int64_t m_first, int lane, uint32_t strips,
                                                             StripColumns& cols) {
#pragma unroll
    for (int s = 0; s < kStrips; ++s) {
        cols.c[s] = -1;
        lds_write_b32(strips + strip_offset(s) + (uint32_t)(4 * lane), 0u);
        lds_write_b32(strips + strip_offset(s) + (uint32_t)(4 * (lane + 64)), 0u);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int64_t n = n_first + lane;
    const int64_t nc = n < a.N ? n : a.N - 1;
    const uint32_t* sc = a.scales + (nc >> 4) * a.KB * kTileRows + (nc & 15);
#pragma unroll 1
    for (int b0 = 0; b0 < a.KB; b0 += 16) {
        uint32_t w[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) w[u] = sc[(int64_t)(b0 + u < a.KB ? b0 + u : a.KB - 1) * kTileRows];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const bool hit = (w[u] & 0x7fff0000u) != 0u && n < a.N && b0 + u < a.KB;
            unsigned long long todo = __builtin_amdgcn_ballot_w64(hit);
            if (todo == 0ull) continue;  // uniform
            if (__builtin_popcountll(todo) > kStrips) return false;  // before anything is fetched
            float x16[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int64_t m = m_first + r * kWave + lane;
                x16[r] = m < a.M ? 16.0f * (float)a.X[m * a.ldx + (int64_t)(b0 + u) * kBlock] : 0.0f;
            }
            while (todo != 0ull) {  // uniform
                const int src = __builtin_ctzll(todo);
                todo &= todo - 1ull;
                // the column's slot, or the first free one (uniform; static indices only)
                int slot = -1;
#pragma unroll
                for (int q = kStrips - 1; q >= 0; --q) slot = cols.c[q] == src ? q : slot;
                if (slot < 0) {
#pragma unroll
                    for (int q = kStrips - 1; q >= 0; --q) slot = cols.c[q] < 0 ? q : slot;
                    if (slot < 0) return false;
#pragma unroll
                    for (int q = 0; q < kStrips; ++q) cols.c[q] = q == slot ? src : cols.c[q];
                }
                const uint32_t word = (uint32_t)__builtin_amdgcn_readlane((int)w[u], src);
                const float dz = f16_bits_to_f32(word & 0xffffu) * f16_bits_to_f32(word >> 16);
#pragma unroll
                for (int r = 0; r < 2; ++r) lds_add_f32(strips + strip_offset(slot) + (uint32_t)(4 * (r * kWave + lane)), dz * x16[r]);
            }
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    return true;
}

// ------------------------------------------------------------------------------------------------
// Workgroup tile 128 (m) x 256 (n), four wavefronts side by side along n, wavefront tile 128 x 64 =
// 4 x 2 v_mfma_f32_32x32x16_f16 (128 accumulator registers per lane), K in quarters of a block
// (64 channels = four MFMA steps), one barrier per quarter.  Two workgroups share a compute unit
// (68 KiB of LDS, about 220 registers), so every SIMD holds two wavefronts from different workgroups:
// one unpacks while the other multiplies, and their barriers are not aligned.
// (A 256 x 256 tile with eight wavefronts, one workgroup per compute unit, was measured too: within
// 3 % where tiles are plentiful, up to 40 % slower where they are not.)
//
// A lane of the 32x32x16 product supplies, for its column n, eight consecutive channels k' of the
// step -- and one low-plane word of the packed tile holds exactly the 16 channels of one step of one
// row, in k' order after the unpack (pairs (slot j, slot j+8)).  So a lane needs, per quarter, the
// four words (16 bytes) of each of its two rows, turns its half of a word into four half2 values
// d (c - 1) in registers, and feeds the matrix core; no dequantized tile is ever stored.
//
// Every operand is copied global -> LDS by the memory pipe itself (buffer_load ... lds: no registers,
// no LDS store instructions), two to three quarters ahead of the arithmetic -- about 1.5 us of lead,
// which covers an HBM miss.
//
// LDS (68 KiB):
//   activations  ring of 3 quarters x 128 rows x 128 bytes, no padding (one copy instruction writes
//                1 KiB = 8 rows, lane l the 16-byte piece l of it).  To keep the 16-byte fragment
//                reads conflict-free, piece p of row r holds channel chunk p ^ swz(r),
//                swz(r) = (r & 7) ^ ((r >> 3) & 1): sixteen consecutive rows reading the same chunk
//                touch sixteen different 16-byte groups of 256 bytes, eight rows eight groups of 128.
//   weights      ring of 4 quarters x 4 wavefronts x 1 KiB: lane (l32, kg) copies the 16 bytes of ITS
//                row j = kg, and later reads both rows (its own piece and that of lane (l32, 1 - kg)).
//                Private to the wavefront: ordered by the load counter alone, no barrier.
//   scales       ring of 4 quarters x 4 wavefronts x 256 bytes, same pattern with 4 bytes per lane.
// The weight ring runs one quarter further ahead than the activation ring because the last MFMA step
// of a quarter already unpacks the first words of the next one.
//
// All LDS reads are written as inline instructions with their own counter waits: the compiler orders
// every LDS read it can see after ALL outstanding global -> LDS copies, which would drain the
// look-ahead at the first read of each quarter.  Since no load returns into registers, it inserts no
// load-counter waits of its own inside the loop either; the explicit ones are all there are.
//
// Tile order: workgroups are dealt to the 8 chiplets round-robin by the hardware, so chiplet x takes
// the contiguous run [x * per, (x+1) * per) of the tile list.  The list walks panels of four tile
// rows (512 activation rows), inside a panel column by column: the workgroups that run together on
// one chiplet then cover 4 x 16 tiles and share, in that chiplet's L2, four activation slabs (the
// expensive operand: 2 bytes per element) among sixteen workgroups each and sixteen weight slabs
// (0.39 bytes per element) among four.
constexpr int GM = 128, GN = 256, GK = 64;
constexpr int GT = 256;  // threads
constexpr int kXStages = 3, kWStages = 4;
constexpr int kXStageBytes = GM * GK * 2;                   // 16384
constexpr int kWRingBase = kXStages * kXStageBytes;         // 49152
constexpr int kWStageBytes = 4 * 1024;                      // 4 wavefronts x 64 lanes x 16 bytes
constexpr int kSRingBase = kWRingBase + kWStages * kWStageBytes;  // 65536
constexpr int kSStageBytes = 4 * 256;                       // 4 wavefronts x 64 lanes x 4 bytes
constexpr int kGemmLds = kSRingBase + kWStages * kSStageBytes;    // 69632
constexpr int kPanel = 4;                                   // tile rows per panel

template <int OFF>
__device__ __forceinline__ half8 lds_read_b128(uint32_t addr) {
    half8 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_read_u4(uint32_t addr) {
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}
template <int OFF>
__device__ __forceinline__ uint32_t lds_read_b32(uint32_t addr) {
    uint32_t r;
    asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}
// wait until at most N LDS reads are outstanding; the values are passed through so that no use of
// them can be scheduled ahead of the wait
#define ITQ3S_LDS_WAIT(N, af) asm volatile("s_waitcnt lgkmcnt(" #N ")" : "+v"(af[0]), "+v"(af[1]), "+v"(af[2]), "+v"(af[3]))

// Position of tile t in the walk described above.
__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int panel = t / (kPanel * tiles_n), within = t - panel * (kPanel * tiles_n);
    const int rows = tiles_m - panel * kPanel < kPanel ? tiles_m - panel * kPanel : kPanel;  // the last panel may be short
    tn = within / rows;
    tm = panel * kPanel + (within - tn * rows);
}

// Store 32 rows (m_first ..) of a wavefront's 64 columns (n0 + 64 wn ..).  Accumulator register v of a
// 32x32 block: row = 8*(v/4) + 4*(lane/32) + v%4, column = lane%32.  kTerms: minus the zero-point
// terms of these rows, from registers (1) or from a few columns' strips in LDS, whose row of m_first is row0 (2).
// Bound by instructions, fetched once each: 128 stores a lane in straight-line code.  With the output type asked
// for and a 64-bit row product at every store (14 instructions), the wavefronts of a second, partly filled round
// came up to each other's delay and the launch lost what the shorter main loop had gained: K x N = 1024x11008, M = 2048,
// fp16, one block in a thousand with a zero-point 74.5 us; with the type as a template and one pointer moved
// from row to row 59.1 (without zero-points 58.2 -> 53.5).
template <int kTerms, typename Out>
__device__ __forceinline__ void store_rows_as(const GemmArgs& a, const floatx16 (&acc)[2], int64_t m_first, int64_t n0, int wn, int lane,
                                           const floatx16 (*in_regs)[2] = nullptr, int row0 = 0, uint32_t strips = 0, const StripColumns* cols = nullptr) {
    const int l32 = lane & 31, kg = lane >> 5;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t n = n0 + wn * 64 + j * 32 + l32;
        floatx16 terms;
        if constexpr (kTerms == 1) terms = (*in_regs)[j];
        if constexpr (kTerms == 2) {
            const int col = 32 * j + l32;
            int slot = -1;
#pragma unroll
            for (int q = 0; q < kStrips; ++q) slot = cols->c[q] == col ? q : slot;
            // sixteen reads in flight, one wait
            uint32_t t[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row0 + 8 * (v >> 2) + 4 * kg + (v & 3);
                const uint32_t addr = strips + strip_offset(slot < 0 ? 0 : slot) + (uint32_t)(4 * row);
                asm volatile("ds_read_b32 %0, %1" : "=v"(t[v]) : "v"(addr) : "memory");
            }
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]), "+v"(t[8]), "+v"(t[9]),
                           "+v"(t[10]), "+v"(t[11]), "+v"(t[12]), "+v"(t[13]), "+v"(t[14]), "+v"(t[15]));
#pragma unroll
            for (int v = 0; v < 16; ++v) terms[v] = slot < 0 ? 0.0f : __builtin_bit_cast(float, t[v]);
        }
        const int rows = a.M - m_first < 32 ? (int)(a.M - m_first) : 32;  // of this block that exist
        Out* dst = reinterpret_cast<Out*>(a.Y) + (m_first + 4 * kg) * a.ldy + n;
        if (n < a.N) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 8 * (v >> 2) + 4 * kg + (v & 3);
                float y = acc[j][v];
                if constexpr (kTerms != 0) y = y - terms[v];
                if (row < rows) *dst = (Out)y;
                dst += (v & 3) == 3 ? 5 * a.ldy : a.ldy;
            }
        }
    }
}

template <int kTerms>
__device__ __forceinline__ void store_rows(const GemmArgs& a, const floatx16 (&acc)[2], int64_t m_first, int64_t n0, int wn, int lane,
                                           const floatx16 (*in_regs)[2] = nullptr, int row0 = 0, uint32_t strips = 0, const StripColumns* cols = nullptr) {
    if (a.y_f16) store_rows_as<kTerms, _Float16>(a, acc, m_first, n0, wn, lane, in_regs, row0, strips, cols);
    else store_rows_as<kTerms, float>(a, acc, m_first, n0, wn, lane, in_regs, row0, strips, cols);
}

// Store a wavefront's 128 x 64 block (rows m0.., columns n0 + 64 wn ..).
__device__ __forceinline__ void store_tile(const GemmArgs& a, const floatx16 (&acc)[4][2], int64_t m0, int64_t n0, int wn, int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i) store_rows<0>(a, acc[i], m0 + i * 32, n0, wn, lane);
}

// (two wavefronts per SIMD: at most 256 registers)
__global__ __launch_bounds__(GT) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_kernel(const GemmGroup group, int tiles_m, int items, int per_chiplet) {
    extern __shared__ __align__(1024) char lds[];
    // LDS byte address of the buffer, for the read instructions below that take raw addresses
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    int item = xcd * per_chiplet + slot;
    if (slot >= per_chiplet || item >= items) return;
    const auto* const kargs = (const __attribute__((address_space(4))) GemmGroup*)__builtin_amdgcn_kernarg_segment_ptr();
    const int ti = (item >= group.t[1].first_item ? 1 : 0) + (item >= group.t[2].first_item ? 1 : 0) + (item >= group.t[3].first_item ? 1 : 0);
    GemmArgs a = group.common;
    a.codes = kargs->t[ti].codes;
    a.scales = kargs->t[ti].scales;
    a.Y = kargs->t[ti].Y;
    a.N = kargs->t[ti].N;
    a.ldy = kargs->t[ti].ldy;
    a.NT = (int)((a.N + 15) >> 4);
    const int tiles_n = kargs->t[ti].tiles_n;
    item -= kargs->t[ti].first_item;
    // the splits of a tile are neighbours in the list
    const int t = item / a.splits, split = item - t * a.splits;
    int tm, tn;
    tile_coords(t, tiles_m, tiles_n, tm, tn);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave;
    const int l32 = lane & 31, kg = lane >> 5;
    const int64_t m0 = (int64_t)tm * GM;
    const int64_t n0 = (int64_t)tn * GN;
    const int KT = (int)(a.K / GK);
    // this workgroup's share of K: whole blocks, quarters q0 .. q1 - 1
    const int q0 = 4 * (int)((int64_t)split * a.KB / a.splits), q1 = 4 * (int)((int64_t)(split + 1) * a.KB / a.splits);

    // All copies go through buffer descriptors: a 32-bit per-lane offset fixed for the whole kernel
    // plus a scalar offset that advances with the stage -- no address arithmetic in the vector pipe.
    // Steps past the end of K repeat the last stage (valid memory, never consumed).
    constexpr int kRsrcFlags = 0x00027000;  // raw buffer, 32-bit elements
    // ---- activations: wavefront w copies pieces 4w .. 4w+3 of a stage (8 rows each); lane l supplies
    // row l/8 of the piece and the chunk that belongs at position l%8 of that row.  Rows past M read
    // row M-1 (their outputs are never stored).
    const __amdgpu_buffer_rsrc_t x_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(a.Xt + m0 * a.K), 0, (int)(GM * a.K * 2), kRsrcFlags);
    int xoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t row = 8 * (4 * wave + i) + (lane >> 3);
        if (m0 + row > a.M - 1) row = a.M - 1 - m0;
        const int chunk = (lane & 7) ^ (lane >> 3) ^ (i & 1);
        xoff[i] = (int)(row * a.K * 2 + chunk * 16);
    }
    // ---- weights: the lane's OWN row n = n0 + wn*64 + kg*32 + l32, as byte offsets from the
    // workgroup's first tile row (16 tile rows x KB tiles: far below 2^31 bytes for any K accepted here)
    const int64_t nt0 = n0 >> 4;
    const int64_t wg_tile_rows = a.NT - nt0 < 16 ? a.NT - nt0 : 16;
    const __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(a.codes + nt0 * a.KB * kTileWords), 0, (int)(wg_tile_rows * a.KB * kTileWords * 4), kRsrcFlags);
    const __amdgpu_buffer_rsrc_t s_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(a.scales + nt0 * a.KB * kTileRows), 0, (int)(wg_tile_rows * a.KB * kTileRows * 4), kRsrcFlags);
    int woff, soff;
    {
        const int r16 = l32 & 15;
        int64_t tr = wn * 4 + (l32 >> 4) + 2 * kg;
        if (nt0 + tr > a.NT - 1) tr = a.NT - 1 - nt0;
        woff = (int)(tr * a.KB * kTileWords + 4 * r16) * 4;  // low-plane words of storage lane 16 q + r16: + 256 q bytes
        soff = (int)(tr * a.KB * kTileRows + r16) * 4;
    }
    auto copy_x = [&](int kt, int ring) {
        const int k_bytes = (kt < KT ? kt : KT - 1) * (GK * 2);
        char* dst = lds + ring * kXStageBytes + 4096 * wave;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (__attribute__((address_space(3))) void*)(dst + 1024 * i), 16, xoff[i], k_bytes, 0, 0);
    };
    auto copy_w = [&](int kt_) {  // quarter kt of the rows: block kt/4, quarter kt%4; ring position kt%4
        const int kt = kt_ < KT ? kt_ : KT - 1;
        const int b = kt >> 2, q = kt & 3, ring = kt_ & 3;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c_rsrc, (__attribute__((address_space(3))) void*)(lds + kWRingBase + ring * kWStageBytes + 1024 * wave),
                                                 16, woff, b * (kTileWords * 4) + 256 * q, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(s_rsrc, (__attribute__((address_space(3))) void*)(lds + kSRingBase + ring * kSStageBytes + 256 * wave),
                                                 4, soff, b * (kTileRows * 4), 0, 0);
    };

    // ---- fragment reads: row i*32 + l32, chunk 2 ks + kg, at position chunk ^ swz(row);
    // swz depends on l32 only, so one byte offset per step ks serves all four i (+ 4096 i)
    uint32_t aoff[4];
    {
        const int s = (l32 & 7) ^ ((l32 >> 3) & 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) aoff[ks] = lds_base + (uint32_t)(l32 * 128 + (((2 * ks + kg) ^ s) * 16));
    }
    const uint32_t wread = lds_base + (uint32_t)(kWRingBase + 1024 * wave + 16 * l32);  // row 0 here, row 1 at + 512
    const uint32_t sread = lds_base + (uint32_t)(kSRingBase + 256 * wave + 4 * l32);    // row 0 here, row 1 at + 128

    uint32_t any_z = 0;
    half2v dd[2];
    auto set_scale = [&](uint32_t s0, uint32_t s1) {
        const _Float16 d0 = __builtin_bit_cast(_Float16, (uint16_t)(s0 & 0xffffu)), d1 = __builtin_bit_cast(_Float16, (uint16_t)(s1 & 0xffffu));
        dd[0] = half2v{d0, d0};
        dd[1] = half2v{d1, d1};
        any_z |= ((s0 | s1) >> 16) & 0x7fffu;
    };
    // Unpack without shifts: the two code bits of pair p sit at bits 2p+1:2p of each half of the
    // word.  OR-ed into the mantissa of the half 2^(10-2p) (bit 2p of whose mantissa weighs exactly 1)
    // they form 2^(10-2p) + c; adding -(2^(10-2p) + 1) gives the digit c - 1 exactly, times d (exact).
    // One and-or, one add, one multiply per pair of weights.
    auto unpack = [&](uint32_t word, int j) -> half8 {
        const uint32_t v = word >> (8 * kg);
        uint32_t o[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            constexpr uint32_t kMagic[4] = {0x64006400u, 0x5C005C00u, 0x54005400u, 0x4C004C00u};  // 1024, 256, 64, 16
            constexpr float kBase[4] = {1024.0f, 256.0f, 64.0f, 16.0f};
            uint32_t bits;
            asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(bits) : "v"(v), "s"(0x00030003u << (2 * p)), "v"(kMagic[p]));
            const _Float16 o1 = (_Float16)(-(kBase[p] + 1.0f));
            half2v h = __builtin_bit_cast(half2v, bits);
            h = (h + half2v{o1, o1}) * dd[j];
            o[p] = __builtin_bit_cast(uint32_t, h);
        }
        const uint4 u = make_uint4(o[0], o[1], o[2], o[3]);
        return __builtin_bit_cast(half8, u);
    };

    floatx16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    half8 bf[2];
    auto step = [&](const half8 (&af)[4], uint32_t nw0, uint32_t nw1) {
        const half8 n0v = unpack(nw0, 0), n1v = unpack(nw1, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[i], bf[j], acc[i][j], 0, 0, 0);
        bf[0] = n0v;
        bf[1] = n1v;
    };
    auto interleave = [&]() {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        }
    };
    half8 af0[4], af1[4];
    auto read_a = [&](uint32_t addr, half8 (&af)[4]) {
        af[0] = lds_read_b128<0>(addr);
        af[1] = lds_read_b128<4096>(addr);
        af[2] = lds_read_b128<8192>(addr);
        af[3] = lds_read_b128<12288>(addr);
    };

    // The loop is rotated by one MFMA step: a trip starts right after a barrier with the LAST step of
    // the previous quarter (its fragments are already in registers), so that the matrix cores have
    // work while the first fragment reads of the new quarter are on their way, then runs steps 0..2
    // of its own quarter and ends with the barrier.  By then every wavefront has read the last
    // fragments of the quarter (they sit in registers), so its buffer is free for the copies issued
    // at the top of the next trip.
    //   trip q:  copies X(q+2), W(q+3) | read A(q,0) | [step (q-1,3)] | read A(q,1), W(q+1) |
    //            step (q,0) | read A(q,2) | step (q,1) | read A(q,3) | step (q,2) | waits, barrier
    // kFirst: there is no previous quarter (bf already holds the operands of step (q,0)).
    auto run_trip = [&](int q, int xr, auto first, const u32x4& c0, const u32x4& c1, u32x4& n0w, u32x4& n1w) {
        constexpr bool kFirst = decltype(first)::value;
        {
            const int xd = xr == 0 ? 2 : xr - 1;  // (q + 2) % 3: held quarter q-1, all of whose reads completed before the barrier
            copy_x(q + 2, xd);
            copy_w(q + 3);  // that slot held quarter q-1, read by this wavefront a trip ago
        }
        const uint32_t wr = wread + (uint32_t)(((q + 1) & 3) * kWStageBytes), sr = sread + (uint32_t)(((q + 1) & 3) * kSStageBytes);
        const uint32_t sb = (uint32_t)(xr * kXStageBytes);
        __builtin_amdgcn_sched_barrier(0);
        read_a(aoff[0] + sb, af0);
        if constexpr (!kFirst) {
            // last step of the previous quarter: fragments in af1 (read before the barrier); unpacks the
            // first words of this quarter, whose scale was set a trip ago
            step(af1, c0.x, c1.x);
            interleave();
            __builtin_amdgcn_sched_barrier(0);
        }
        n0w = lds_read_u4<0>(wr);
        n1w = lds_read_u4<512>(wr);
        uint32_t s0 = lds_read_b32<0>(sr), s1 = lds_read_b32<128>(sr);
        read_a(aoff[1] + sb, af1);
        asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(af0[0]), "+v"(af0[1]), "+v"(af0[2]), "+v"(af0[3]));
        step(af0, c0.y, c1.y);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        read_a(aoff[2] + sb, af0);
        asm volatile("s_waitcnt lgkmcnt(4)"
                     : "+v"(af1[0]), "+v"(af1[1]), "+v"(af1[2]), "+v"(af1[3]), "+v"(n0w), "+v"(n1w), "+v"(s0), "+v"(s1));
        step(af1, c0.z, c1.z);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        read_a(aoff[3] + sb, af1);
        ITQ3S_LDS_WAIT(4, af0);
        step(af0, c0.w, c1.w);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        set_scale(s0, s1);  // for the unpack of the next quarter's first words, at the top of the next trip
        ITQ3S_LDS_WAIT(0, af1);
        // Everything issued before this trip's six copies has landed: the activations of quarter q+1
        // and the weights of quarter q+2 among them (copies complete in order).
        asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };

    // Prologue: quarters 0 and 1 of everything and quarter 2 of the weights, in two groups of six
    // copies, so that waiting for all but six leaves exactly the second group in flight.
    u32x4 wa0, wa1, wb0, wb1;
    copy_x(q0, 0);
    copy_w(q0);
    __builtin_amdgcn_sched_barrier(0);
    copy_x(q0 + 1, 1);
    copy_w(q0 + 1);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    copy_w(q0 + 2);
    __builtin_amdgcn_sched_barrier(0);
    {
        wa0 = lds_read_u4<0>(wread);
        wa1 = lds_read_u4<512>(wread);
        uint32_t s0 = lds_read_b32<0>(sread), s1 = lds_read_b32<128>(sread);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(wa0), "+v"(wa1), "+v"(s0), "+v"(s1));
        set_scale(s0, s1);
        bf[0] = unpack(wa0.x, 0);
        bf[1] = unpack(wa1.x, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(2)" ::: "memory");  // quarter 1 has landed as well; only the two copies of copy_w(2) may be in flight
    __builtin_amdgcn_s_barrier();
    // The two register sets of the weights alternate by name, so trips come in pairs: the first trip
    // on its own, pairs (1,2), (3,4), ..., and the last trip (K is a multiple of 256: the number of
    // quarters is a multiple of four, so it is odd-numbered).
    run_trip(q0, 0, std::true_type{}, wa0, wa1, wb0, wb1);
    int xr = 1;
    for (int q = q0 + 1; q + 1 < q1; q += 2) {
        run_trip(q, xr, std::false_type{}, wb0, wb1, wa0, wa1);
        xr = xr == 2 ? 0 : xr + 1;
        run_trip(q + 1, xr, std::false_type{}, wa0, wa1, wb0, wb1);
        xr = xr == 2 ? 0 : xr + 1;
    }
    run_trip(q1 - 1, xr, std::false_type{}, wb0, wb1, wa0, wa1);
    // last step of the last quarter (the words it unpacks are never used)
    step(af1, wa0.x, wa1.x);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the look-ahead copies past the last quarter still target this workgroup's LDS

    // Format check, apart from the arithmetic: the high plane of the workgroup's 16 tile rows must be
    // zero (128 words per tile, a quarter of the packed bytes, read once more here).
    if (a.flags != nullptr && tm == 0 && split == 0) {  // once per tile column
        const uint4* hp = reinterpret_cast<const uint4*>(a.codes + nt0 * a.KB * kTileWords);
        const int64_t tiles = wg_tile_rows * a.KB;  // 32 pieces of 16 bytes per tile, at word 256 of each
        uint32_t bad = 0;
#pragma unroll 2
        for (int64_t i = tid; i < tiles * 32; i += GT) {
            const uint4 v = hp[(i >> 5) * (kTileWords / 4) + kTileLoWords / 4 + (i & 31)];
            bad |= v.x | v.y | v.z | v.w;
        }
        if (bad != 0u) atomicOr(a.flags, kFlagBadCode);
    }
    const bool zero_points = __builtin_amdgcn_ballot_w64(any_z != 0u) != 0ull;  // did a lane of this wavefront meet one?
    if (a.splits > 1) {
        // split-K: park the sums; the launch that follows adds the shares of every tile in split order
        floatx4* const mine = reinterpret_cast<floatx4*>(a.partial) + ((int64_t)(t * a.splits + split) * 32) * GT + tid;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    mine[((i * 2 + j) * 4 + c) * GT] = floatx4{acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
        if (zero_points && lane == 0) atomicOr(a.zflags + t, 1u);
        return;
    }
    if (zero_points) {
        // (columns past N read clamped rows and may trigger this needlessly; nothing is stored for them)
        {
            // first the cheap way: at most eight columns with zero-points, strips in this wavefront's own
            // corner of the weight ring (its copies have landed; nobody else touches it)
            const uint32_t strips = lds_base + kWRingBase + (uint32_t)wave * 1024u;
            StripColumns cols;
            if (zero_point_terms_few_columns(a, n0 + wn * 64, m0, lane, strips, cols)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) store_rows<2>(a, acc[i], m0 + 32 * i, n0, wn, lane, nullptr, 32 * i, strips, &cols);
                return;
            }
        }
        // otherwise 32 rows at a time in registers
        static_assert(kWStageBytes == 4096 && kWStages * 2 >= kStrips, "two strips of 128 floats in the wavefront's KiB of every stage");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            floatx16 terms[2];
            zero_point_terms(a, n0 + wn * 64, m0 + 32 * i, lane, lds_base + kWRingBase + (uint32_t)wave * 1024u, terms);
            store_rows<1>(a, acc[i], m0 + 32 * i, n0, wn, lane, &terms);
        }
        return;
    }
    store_tile(a, acc, m0, n0, wn, lane);
}

// Second launch of a split-K matmul: four workgroups per tile, one per 32-row slab, add the shares
// in split order (thread and register layout as in the contraction kernel) and finish the slab.
__global__ __launch_bounds__(GT) void gemm_reduce_kernel(const GemmArgs a, int tiles_m, int tiles_n) {
    const int t = (int)(blockIdx.x >> 2), i = (int)(blockIdx.x & 3), tid = threadIdx.x, lane = tid & 63, wn = tid >> 6;
    int tm, tn;
    tile_coords(t, tiles_m, tiles_n, tm, tn);
    const floatx4* const all = reinterpret_cast<const floatx4*>(a.partial) + ((int64_t)t * a.splits * 32) * GT + tid;
    floatx16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int piece = (i * 2 + j) * 4 + c;
            floatx4 share[kGemmMaxSplits];  // all loads first (absent splits re-read share 0), then the sum in split order
#pragma unroll
            for (int sp = 0; sp < kGemmMaxSplits; ++sp) share[sp] = all[((int64_t)(sp < a.splits ? sp : 0) * 32 + piece) * GT];
            floatx4 sum = share[0];
#pragma unroll
            for (int sp = 1; sp < kGemmMaxSplits; ++sp)
                if (sp < a.splits) sum = sum + share[sp];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][4 * c + e] = sum[e];
        }
    const int64_t m_first = (int64_t)tm * GM + i * 32, n0 = (int64_t)tn * GN;
    if (a.zflags[t] != 0u) {
        __shared__ __align__(16) float row_values[4][32];  // of each wavefront
        floatx16 terms[2];
        zero_point_terms(a, n0 + wn * 64, m_first, lane, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)row_values[wn], terms);
        store_rows<1>(a, acc, m_first, n0, wn, lane, &terms);
        return;
    }
    store_rows<0>(a, acc, m_first, n0, wn, lane);
}

// Splits of K per tile, each at least four blocks long, when the tiles alone leave half of the chip idle.  A
// workgroup alone on a compute unit does nearly the work of two that share it, and every share costs its
// way through memory twice, so one workgroup per unit is the aim where the tiles divide the units well and K
// is not so long that the shares do not count; else two per unit.  One / two per unit, 512 rows, us: 11008x4096
// 63 / 72, 14336x4096 75 / 83, 8192x8192 79 / 83, but 28672x8192 232 / 223; 14336x4096 with 700 rows (96
// tiles: 192 or 480 workgroups) 109 / 104.  A function of the shape only.
int gemm_splits(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + GM - 1) / GM) * ((N + GN - 1) / GN);
    if (tiles > kGemmSplitMaxTiles) return 1;
    int64_t s = 256 / tiles;
    if (K > 20480 || s * tiles < 208) s = 512 / tiles;
    if (s > kGemmMaxSplits) s = kGemmMaxSplits;
    if (s > K / kBlock / 4) s = K / kBlock / 4;
    return s < 1 ? 1 : (int)s;
}
size_t gemm_partial_bytes(int64_t M, int64_t N, int64_t K) {
    const int s = gemm_splits(M, N, K);
    return s > 1 ? (size_t)s * (size_t)(((M + GM - 1) / GM) * ((N + GN - 1) / GN)) * (GM * GN * 4) : 0;
}

int launch_gemm(const GemvWeight* w, int count, int64_t K, const _Float16* Xt, const _Float16* X, int64_t ldx, int64_t M, int y_f16, float* partial,
                size_t partial_bytes, uint32_t* zflags, uint32_t* flags, hipStream_t stream) {
    const int64_t tiles_m = (M + GM - 1) / GM;
    if (K > kGemmMaxK) return -2;
    static DeviceOnce lds_limit;
    if (!raise_lds_limit(lds_limit, reinterpret_cast<const void*>(gemm_kernel), kGemmLds)) return -6;
    GemmGroup group;
    GemmArgs& a = group.common;
    a.codes = nullptr; a.scales = nullptr; a.Y = nullptr; a.N = 0; a.ldy = 0; a.NT = 0;
    a.Xt = Xt; a.X = X; a.ldx = ldx; a.flags = flags; a.K = K; a.M = M; a.KB = (int)(K / kBlock); a.y_f16 = y_f16;
    a.partial = partial; a.zflags = zflags;
    int64_t items = 0;
    int n = 0;
    auto add = [&](const GemvWeight& v) {
        group.t[n++] = GemmTensor{v.codes, v.scales, v.Y, v.N, v.ldy, (int)items, (int)((v.N + GN - 1) / GN)};
        items += tiles_m * ((v.N + GN - 1) / GN) * a.splits;
    };
    auto launch = [&]() -> int {
        if (items >= 0x7fffffff / 8) return -2;
        for (int i = n; i < kGemvMaxGroup; ++i) {
            group.t[i] = group.t[0];
            group.t[i].first_item = 0x7fffffff;
        }
        const int per = (int)((items + 7) / 8);
        const dim3 g((unsigned)(per * 8));
        const LaunchTiming tm = take_launch_timing();
        if (tm.start != nullptr) hipExtLaunchKernelGGL(gemm_kernel, g, dim3(GT), kGemmLds, stream, tm.start, tm.stop, 0, group, (int)tiles_m, (int)items, per);
        else hipLaunchKernelGGL(gemm_kernel, g, dim3(GT), kGemmLds, stream, group, (int)tiles_m, (int)items, per);
        return hipGetLastError() == hipSuccess ? 0 : -6;
    };
    // a tensor that splits K has a launch of its own (the room for shares is one tensor's), and only if the
    // caller's workspace has room for its shares (a grouped call sizes it for its largest tensor)
    auto splits_of = [&](const GemvWeight& v) {
        return partial != nullptr && zflags != nullptr && gemm_partial_bytes(M, v.N, K) <= partial_bytes ? gemm_splits(M, v.N, K) : 1;
    };
    a.splits = 1;
    for (int i = 0; i < count; ++i)
        if (splits_of(w[i]) == 1) add(w[i]);
    if (n > 0) {
        const int rc = launch();
        if (rc != 0) return rc;
    }
    for (int i = 0; i < count; ++i) {
        a.splits = splits_of(w[i]);
        if (a.splits == 1) continue;
        n = 0;
        items = 0;
        add(w[i]);
        const int rc = launch();
        if (rc != 0) return rc;
        GemmArgs r = a;
        r.codes = w[i].codes; r.scales = w[i].scales; r.Y = w[i].Y; r.N = w[i].N; r.ldy = w[i].ldy; r.NT = (int)((w[i].N + 15) / 16);
        const int tiles_n = (int)((w[i].N + GN - 1) / GN);
        hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)(tiles_m * tiles_n * 4)), dim3(GT), 0, stream, r, (int)tiles_m, tiles_n);
        if (hipGetLastError() != hipSuccess) return -6;
    }
    return 0;
}

}  // namespace itq3s
