// C-ABI entry points of libitq3s: argument validation on the host, then launches.  See
// include/itq3s.h for the contract of every call (include/itq3s_bench.h for the measurement aids).
#include "../../include/itq3s.h"
#include "../../include/itq3s_bench.h"
#include "itq3s_kernels.h"

#include <atomic>
#include <mutex>

// Scratch of itq3s_matmul_static: one array per device the library runs on, held until the process
// ends.  The name below is a host-side stand-in for the symbol; device code gets the address that
// hipGetSymbolAddress returns for the current device (scratch_of_current_device).
static __device__ __align__(256) unsigned char scratch[ITQ3S_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

// Address of `scratch` on the current device (looked up once per device), or null.
void* scratch_of_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p != nullptr) return p;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (p == nullptr) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return nullptr;
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    return p;
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline int pad_m(int64_t M) {
    int mp = 1;
    while (mp < M) mp <<= 1;
    return mp;
}

constexpr int64_t kChunkedMaxM = 2 * itq3s::kGemvMaxM;  // up to here M > 16 may run as two passes of the streaming kernel
constexpr int64_t kSubStreamingMaxM = 64;               // sub-block variant: up to here passes of four rows, the tiled weight-side kernel above

// The streaming kernel for up to 16 rows: what it takes in front of itself, see launch_rotate_frag.
struct FragPlan {
    size_t xt_bytes, total;  // rotated activations (then two sums per block and row); all of it
};
FragPlan plan_frag(int64_t M, int64_t K) {
    if (M <= itq3s::kGemvFusedMaxM) return FragPlan{0, 256};  // it rotates the activations itself: nothing to park
    const int64_t rows = pad_m(M);
    const size_t xt = round_up((size_t)rows * (size_t)K * 2, 256);
    return FragPlan{xt, xt + round_up((size_t)rows * (size_t)(K / 256) * 8, 256) + 256};
}

// The least room that a call is accepted with (the largest over its tensors).  Above 32 rows it is what a kernel with
// fp16 operands once needed, shares of K for few output tiles among it: callers have kept such sizes, and what was
// refused stays refused.  Every such room holds a pass of 16 rows, at least.
size_t least_workspace(int64_t M, int64_t N, int64_t K) {
    if (M <= kChunkedMaxM) return plan_frag(M < itq3s::kGemvMaxM ? M : itq3s::kGemvMaxM, K).total;
    const int64_t tiles = ((M + 127) / 128) * ((N + 255) / 256);
    int64_t shares = 1;
    if (tiles <= 128) {
        shares = 256 / tiles;
        if (K > 20480 || shares * tiles < 208) shares = 512 / tiles;
        if (shares > 8) shares = 8;
        if (shares > K / 1024) shares = K / 1024;
    }
    const size_t partial = shares > 1 ? (size_t)shares * (size_t)tiles * (128 * 256 * 4) : 0;
    return round_up((size_t)M * (size_t)K * 2, 256) + 512 + partial + 256;
}

// Passes of the streaming kernel for 16 rows, two of them: where the many-row kernel's rule leaves a call of up to 32 rows
// to them (17 rows of a thin tensor with long K, more than 32 MB of rotated activations: K above 250,000).  Three: where
// 32 rows of the block-scaled operand would not fit the static scratch that such a call has always fitted.
inline bool passes_of_16(int64_t M, int64_t N, int64_t K) {
    return M <= kChunkedMaxM ? !itq3s::rows_path(M, N, K) : M < 38 && itq3s::mx_bytes(1, K) > (size_t)ITQ3S_STATIC_SCRATCH_BYTES;
}

// Scratch of the kernels for more rows, the same for every tensor of a call: the many-row kernel, the block-scaled ones.
size_t rows_workspace(int64_t M, int64_t K) { return round_up(itq3s::rows_xt_bytes(M, K), 256) + round_up(itq3s::rows_x0_bytes(M, K), 256); }

// The block-scaled kernels over the tensors that each of them takes, in as many slabs of rows as the room asks for (a
// row's results do not depend on the others).  The room holds 32 rows.
int launch_mx_routes(const itq3s_weight* w, const itq3s::Route* route, int count, int64_t K, const _Float16* X, int64_t M, int64_t ldx, int y_f16,
                     unsigned char* Xm, size_t room, uint32_t* flags, hipStream_t st) {
    int64_t slab = M;
    if (room < itq3s::mx_bytes(M, K)) {
        const int64_t most = (int64_t)(room / itq3s::mx_bytes(1, K)) * itq3s::kMxRows, slabs = (M + most - 1) / most;
        slab = ((M + slabs - 1) / slabs + itq3s::kMxRows - 1) / itq3s::kMxRows * itq3s::kMxRows;
    }
    const size_t y_bytes = y_f16 ? 2 : 4;
    for (int64_t m0 = 0; m0 < M; m0 += slab) {
        const int64_t rows = M - m0 < slab ? M - m0 : slab;
        int rc = itq3s::launch_rotate_mx(X + m0 * ldx, rows, K, ldx, Xm, flags, st);
        for (const itq3s::Route r : {itq3s::Route::shares8, itq3s::Route::shares4, itq3s::Route::tiled}) {
            itq3s::GemvWeight gw[ITQ3S_MAX_GROUP];
            int n = 0;
            for (int i = 0; i < count; ++i)
                if (route[i] == r) gw[n++] = itq3s::GemvWeight{w[i].codes, w[i].scales, w[i].N, static_cast<unsigned char*>(w[i].Y) + (size_t)m0 * (size_t)w[i].ldy * y_bytes, w[i].ldy};
            if (rc != 0 || n == 0) continue;
            if (r == itq3s::Route::tiled) rc = itq3s::launch_gemm(gw, n, K, rows, Xm, y_f16, flags, st);
            else rc = itq3s::launch_mx_shares(gw, n, K, rows, Xm, r == itq3s::Route::shares8 ? 8 : 4, y_f16, flags, st);
        }
        if (rc != 0) return rc;
    }
    return 0;
}

}  // namespace

namespace {
// a call with a pair of events armed for the contraction kernel's dispatch, then a wait
template <typename Call>
int timed(float* kernel_ms, Call call) {
    if (!kernel_ms) return ITQ3S_ERR_NULL;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess) return ITQ3S_ERR_LAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return ITQ3S_ERR_LAUNCH;
    }
    itq3s::set_launch_timing(e0, e1);
    int rc = call();
    const bool taken = itq3s::take_launch_timing().start == nullptr;  // (also disarms if validation returned before any launch)
    if (rc == ITQ3S_OK && taken) {
        if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(kernel_ms, e0, e1) != hipSuccess) rc = ITQ3S_ERR_LAUNCH;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}
}  // namespace

extern "C" {

size_t itq3s_codes_bytes(int64_t N, int64_t K) {
    if (N <= 0 || K <= 0 || K % 256 != 0) return 0;
    return (size_t)((N + 15) / 16) * (size_t)(K / 256) * 1536u;
}

size_t itq3s_scales_bytes(int64_t N, int64_t K) {
    if (N <= 0 || K <= 0 || K % 256 != 0) return 0;
    return (size_t)((N + 15) / 16) * (size_t)(K / 256) * 64u;
}

size_t itq3s_matmul_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 0 || N <= 0 || K <= 0 || K % 256 != 0) return 256;
    // room for the kernel that computes the call, and for those that one with less room falls back to
    const size_t least = least_workspace(M, N, K);
    if (M <= itq3s::kGemvMaxM || passes_of_16(M, N, K)) return least;
    const size_t want = itq3s::many_row_route(M, N, K) == itq3s::Route::rows ? rows_workspace(M, K) : itq3s::mx_bytes(M, K);
    return want > least ? want : least;
}

int itq3s_quantize(const float* W, int64_t N, int64_t K, int64_t ldw, uint32_t* codes, uint32_t* scales, uint32_t* status_flags,
                   void* stream) {
    if (!W || !codes || !scales) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || K % 256 != 0 || ldw < K) return ITQ3S_ERR_SHAPE;
    if (((N + 15) / 16) * (K / 256) > 0x3fffffffLL) return ITQ3S_ERR_SHAPE;  // two workgroups per tile, 32-bit grid
    if (!aligned(W, 16) || ldw % 4 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_quantize(W, N, K, ldw, codes, scales, nullptr, status_flags, static_cast<hipStream_t>(stream));
}

int itq3s_roundtrip(const float* W, int64_t N, int64_t K, int64_t ldw, int block_size, uint8_t* codes_out, uint32_t* scales_out,
                    float* W_hat, int64_t ldo, double* err2, uint32_t* status_flags, void* stream) {
    if (!W) return ITQ3S_ERR_NULL;
    if (block_size != 32 && block_size != 64 && block_size != 128 && block_size != 256 && block_size != 512) return ITQ3S_ERR_SHAPE;
    if (N <= 0 || K <= 0 || K % block_size != 0 || ldw < K || (W_hat && ldo < K)) return ITQ3S_ERR_SHAPE;
    if (N > 0x7fffffffLL / ((K + 1023) / 1024)) return ITQ3S_ERR_SHAPE;  // one wavefront per 1024 channels of a row
    if (!aligned(W, 16) || ldw % 4 != 0 || (codes_out && !aligned(codes_out, 16)) || (scales_out && !aligned(scales_out, 4)) ||
        (W_hat && (!aligned(W_hat, 16) || ldo % 4 != 0)) || (err2 && !aligned(err2, 8)) || (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_roundtrip(W, N, K, ldw, block_size, codes_out, scales_out, W_hat, ldo, err2, status_flags,
                                   static_cast<hipStream_t>(stream));
}

int itq3s_dequantize(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, void* W_out, int out_dtype, int64_t ldo,
                     uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !W_out) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || K % 256 != 0 || ldo < K) return ITQ3S_ERR_SHAPE;
    if (((N + 15) / 16) * (K / 256) > 0x7fffffffLL) return ITQ3S_ERR_SHAPE;
    if (out_dtype != ITQ3S_F32 && out_dtype != ITQ3S_F16) return ITQ3S_ERR_DTYPE;
    if (!aligned(W_out, 16) || ldo % 4 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_dequantize(codes, scales, nullptr, N, K, W_out, out_dtype == ITQ3S_F16, ldo, status_flags, static_cast<hipStream_t>(stream));
}

int itq3s_matmul_grouped(const itq3s_weight* w, int count, int64_t K, const void* X, int64_t M, int64_t ldx, int y_dtype, void* workspace,
                         size_t workspace_bytes, uint32_t* status_flags, void* stream) {
    if (!w || !X) return ITQ3S_ERR_NULL;
    if (count < 1 || count > ITQ3S_MAX_GROUP) return ITQ3S_ERR_SHAPE;
    if (K <= 0 || M <= 0 || K % 256 != 0 || ldx < K) return ITQ3S_ERR_SHAPE;
    if (y_dtype != ITQ3S_F32 && y_dtype != ITQ3S_F16) return ITQ3S_ERR_DTYPE;
    if (M > 0x7fffffffLL / (K / 256)) return ITQ3S_ERR_SHAPE;
    if (M > itq3s::kGemvMaxM && K > (1LL << 22)) return ITQ3S_ERR_SHAPE;  // the tiled kernel's 32-bit byte offsets
    if (K > (1LL << 28) || (M <= itq3s::kGemvFusedMaxM && (M - 1) * ldx + K > (1LL << 29))) return ITQ3S_ERR_SHAPE;  // 32-bit byte offsets of the streaming kernel
    size_t need = 0;
    for (int i = 0; i < count; ++i) {
        if (!w[i].codes || !w[i].scales || !w[i].Y) return ITQ3S_ERR_NULL;
        if (w[i].N <= 0 || w[i].ldy < w[i].N || (w[i].N + 15) / 16 > 0x7fffffffLL / (K / 256)) return ITQ3S_ERR_SHAPE;
        if (!aligned(w[i].codes, 16) || !aligned(w[i].scales, 16) || !aligned(w[i].Y, y_dtype == ITQ3S_F16 ? 2 : 4)) return ITQ3S_ERR_ALIGN;
        const size_t need_i = least_workspace(M, w[i].N, K);
        if (need_i > need) need = need_i;
    }
    if (!aligned(X, 16) || ldx % 8 != 0 || (status_flags && !aligned(status_flags, 4))) return ITQ3S_ERR_ALIGN;
    if (!workspace || workspace_bytes < need) return ITQ3S_ERR_WORKSPACE;
    if (!aligned(workspace, 256)) return ITQ3S_ERR_ALIGN;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const _Float16* const Xh = static_cast<const _Float16*>(X);
    const int y_f16 = y_dtype == ITQ3S_F16;
    unsigned char* const base = static_cast<unsigned char*>(workspace);
    if (M <= itq3s::kGemvMaxM) {
        itq3s::GemvWeight gw[ITQ3S_MAX_GROUP];
        for (int i = 0; i < count; ++i) gw[i] = itq3s::GemvWeight{w[i].codes, w[i].scales, w[i].N, w[i].Y, w[i].ldy};
        if (M <= itq3s::kGemvFusedMaxM) return itq3s::launch_gemv(gw, count, K, Xh, ldx, M, y_f16, status_flags, st);
        const int MP = pad_m(M) < 8 ? 8 : pad_m(M);
        _Float16* const Xt = static_cast<_Float16*>(workspace);
        float* const S = reinterpret_cast<float*>(base + plan_frag(M, K).xt_bytes);
        const int rc = itq3s::launch_rotate_frag(Xh, M, K, ldx, MP, Xt, S, status_flags, st);
        if (rc != 0) return rc;
        return itq3s::launch_gemv_rows(gw, count, K, Xt, S, M, MP, y_f16, status_flags, st);
    }
    // More rows: every tensor by the kernel that its own sizes ask for; those of one kernel share a launch, and the kernels
    // follow each other in the same scratch (same stream).  With less room than a kernel takes (a workspace sized for
    // another M, or by an older rule) the many-row kernel's tensors go to the block-scaled one, which takes the rows
    // in slabs; what has no room for 32 rows, and up to 32 rows with too little, goes through passes of 16.
    itq3s_weight mx[ITQ3S_MAX_GROUP], pass[ITQ3S_MAX_GROUP];
    itq3s::Route mx_route[ITQ3S_MAX_GROUP];
    itq3s::GemvWeight rows[ITQ3S_MAX_GROUP];
    int n_rows = 0, n_mx = 0, n_pass = 0;
    const bool room_rows = workspace_bytes >= rows_workspace(M, K);
    const bool room_mx = workspace_bytes >= itq3s::mx_bytes(1, K);
    for (int i = 0; i < count; ++i) {
        if (passes_of_16(M, w[i].N, K)) {
            pass[n_pass++] = w[i];
            continue;
        }
        itq3s::Route r = itq3s::many_row_route(M, w[i].N, K);
        if (r == itq3s::Route::rows && room_rows) {
            rows[n_rows++] = itq3s::GemvWeight{w[i].codes, w[i].scales, w[i].N, w[i].Y, w[i].ldy};
            continue;
        }
        if (!room_mx || (r == itq3s::Route::rows && M <= kChunkedMaxM)) {
            pass[n_pass++] = w[i];
            continue;
        }
        mx_route[n_mx] = r == itq3s::Route::rows ? itq3s::Route::shares8 : r;
        mx[n_mx++] = w[i];
    }
    int rc = 0;
    if (n_rows > 0)
        rc = itq3s::launch_rows(rows, n_rows, K, Xh, ldx, M, reinterpret_cast<_Float16*>(base),
                                reinterpret_cast<_Float16*>(base + round_up(itq3s::rows_xt_bytes(M, K), 256)), y_f16, status_flags, st);
    if (rc == 0 && n_pass > 0) {
        const size_t y_bytes = y_f16 ? 2 : 4;
        for (int64_t m0 = 0; m0 < M && rc == 0; m0 += itq3s::kGemvMaxM) {
            itq3s_weight part[ITQ3S_MAX_GROUP];
            for (int i = 0; i < n_pass; ++i) {
                part[i] = pass[i];
                part[i].Y = static_cast<unsigned char*>(pass[i].Y) + (size_t)m0 * (size_t)pass[i].ldy * y_bytes;
            }
            const int64_t m = M - m0 < itq3s::kGemvMaxM ? M - m0 : itq3s::kGemvMaxM;
            rc = itq3s_matmul_grouped(part, n_pass, K, Xh + m0 * ldx, m, ldx, y_dtype, workspace, workspace_bytes, status_flags, stream);
        }
    }
    if (rc == 0 && n_mx > 0) rc = launch_mx_routes(mx, mx_route, n_mx, K, Xh, M, ldx, y_f16, base, workspace_bytes, status_flags, st);
    return rc;
}

int itq3s_matmul(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, const void* X, int64_t M, int64_t ldx, void* Y,
                 int y_dtype, int64_t ldy, void* workspace, size_t workspace_bytes, uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !X || !Y) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || M <= 0 || K % 256 != 0 || ldx < K || ldy < N) return ITQ3S_ERR_SHAPE;
    const itq3s_weight w = {codes, scales, N, Y, ldy};
    return itq3s_matmul_grouped(&w, 1, K, X, M, ldx, y_dtype, workspace, workspace_bytes, status_flags, stream);
}

// ---- the sub-block-scale variant of the format (116 bytes per block)

size_t itq3s_subscales_bytes(int64_t N, int64_t K) {
    if (N <= 0 || K <= 0 || K % 256 != 0) return 0;
    return (size_t)((N + 15) / 16) * (size_t)(K / 256) * 256u;
}

int itq3s_quantize_sub(const float* W, int64_t N, int64_t K, int64_t ldw, uint32_t* codes, uint32_t* scales, uint32_t* subscales,
                       uint32_t* status_flags, void* stream) {
    if (!subscales) return ITQ3S_ERR_NULL;
    if (!aligned(subscales, 16)) return ITQ3S_ERR_ALIGN;
    if (!W || !codes || !scales) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || K % 256 != 0 || ldw < K) return ITQ3S_ERR_SHAPE;
    if (((N + 15) / 16) * (K / 256) > 0x3fffffffLL) return ITQ3S_ERR_SHAPE;
    if (!aligned(W, 16) || ldw % 4 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_quantize(W, N, K, ldw, codes, scales, subscales, status_flags, static_cast<hipStream_t>(stream));
}

int itq3s_dequantize_sub(const uint32_t* codes, const uint32_t* scales, const uint32_t* subscales, int64_t N, int64_t K, void* W_out,
                         int out_dtype, int64_t ldo, uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !subscales || !W_out) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || K % 256 != 0 || ldo < K) return ITQ3S_ERR_SHAPE;
    if (((N + 15) / 16) * (K / 256) > 0x7fffffffLL) return ITQ3S_ERR_SHAPE;
    if (out_dtype != ITQ3S_F32 && out_dtype != ITQ3S_F16) return ITQ3S_ERR_DTYPE;
    if (!aligned(W_out, 16) || ldo % 4 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || !aligned(subscales, 16) ||
        (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_dequantize(codes, scales, subscales, N, K, W_out, out_dtype == ITQ3S_F16, ldo, status_flags, static_cast<hipStream_t>(stream));
}

int itq3s_matmul_sub(const uint32_t* codes, const uint32_t* scales, const uint32_t* subscales, int64_t N, int64_t K, const void* X, int64_t M,
                     int64_t ldx, void* Y, int y_dtype, int64_t ldy, void* workspace, size_t workspace_bytes, uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !subscales || !X || !Y) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || M <= 0 || K % 256 != 0 || ldx < K || ldy < N) return ITQ3S_ERR_SHAPE;
    if (K > (1LL << 28) || 3 * ldx + K > (1LL << 29) || (N + 15) / 16 > 0x7fffffffLL / (K / 256)) return ITQ3S_ERR_SHAPE;
    if (y_dtype != ITQ3S_F32 && y_dtype != ITQ3S_F16) return ITQ3S_ERR_DTYPE;
    if (!aligned(X, 16) || ldx % 8 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || !aligned(subscales, 16) ||
        !aligned(Y, y_dtype == ITQ3S_F16 ? 2 : 4) || (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int y_f16 = y_dtype == ITQ3S_F16;
    // many rows: the tiled kernel that reconstructs weight tiles on chip (one pass over the weights per 512 rows)
    if (M > kSubStreamingMaxM) {
        if ((M + 511) / 512 > 65535) return ITQ3S_ERR_SHAPE;
        return itq3s::launch_gemm_weight_side(codes, scales, subscales, N, K, static_cast<const _Float16*>(X), ldx, M, Y, y_f16, ldy, status_flags, st);
    }
    // the streaming kernel: passes of up to 16 rows; a pass of up to four rows (eight for small tensors) rotates
    // the activations itself, a longer one takes them from a rotation launch through the workspace
    const FragPlan p = plan_frag(M < itq3s::kGemvMaxM ? M : itq3s::kGemvMaxM, K);
    if (M > itq3s::kGemvFusedMaxM) {
        if (!workspace || workspace_bytes < p.total) return ITQ3S_ERR_WORKSPACE;
        if (!aligned(workspace, 256)) return ITQ3S_ERR_ALIGN;
    }
    const size_t y_bytes = y_f16 ? 2 : 4;
    for (int64_t m0 = 0; m0 < M; m0 += itq3s::kGemvMaxM) {
        const int64_t rows = M - m0 < itq3s::kGemvMaxM ? M - m0 : itq3s::kGemvMaxM;
        const _Float16* Xh = static_cast<const _Float16*>(X) + m0 * ldx;
        itq3s::GemvWeight gw{codes, scales, N, static_cast<unsigned char*>(Y) + (size_t)m0 * (size_t)ldy * y_bytes, ldy, subscales};
        int rc;
        if (itq3s::gemv_sub_fused(rows, N, K, ldx)) {
            rc = itq3s::launch_gemv(&gw, 1, K, Xh, ldx, rows, y_f16, status_flags, st);
        } else {
            const int MP = pad_m(rows) < 8 ? 8 : pad_m(rows);
            _Float16* Xt = static_cast<_Float16*>(workspace);
            float* S = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + p.xt_bytes);
            rc = itq3s::launch_rotate_frag(Xh, rows, K, ldx, MP, Xt, S, status_flags, st);
            if (rc == 0) rc = itq3s::launch_gemv_rows(&gw, 1, K, Xt, S, rows, MP, y_f16, status_flags, st);
        }
        if (rc != 0) return rc;
    }
    return ITQ3S_OK;
}

int itq3s_matmul_static(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, const void* X, int64_t M, int64_t ldx, void* Y,
                        int y_dtype, int64_t ldy, uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !X || !Y) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || M <= 0 || K % 256 != 0 || ldx < K || ldy < N) return ITQ3S_ERR_SHAPE;
    if (least_workspace(M, N, K) > (size_t)ITQ3S_STATIC_SCRATCH_BYTES) return ITQ3S_ERR_WORKSPACE;
    void* ws = scratch_of_current_device();
    if (ws == nullptr) return ITQ3S_ERR_LAUNCH;
    return itq3s_matmul(codes, scales, N, K, X, M, ldx, Y, y_dtype, ldy, ws, (size_t)ITQ3S_STATIC_SCRATCH_BYTES, status_flags, stream);
}

int itq3s_matmul_weight_side(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, const void* X, int64_t M, int64_t ldx,
                             void* Y, int y_dtype, int64_t ldy, uint32_t* status_flags, void* stream) {
    if (!codes || !scales || !X || !Y) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || M <= 0 || K % 256 != 0 || ldx < K || ldy < N) return ITQ3S_ERR_SHAPE;
    if ((N + 15) / 16 > 0x7fffffffLL / (K / 256) || (M + 511) / 512 > 65535) return ITQ3S_ERR_SHAPE;
    if (y_dtype != ITQ3S_F32 && y_dtype != ITQ3S_F16) return ITQ3S_ERR_DTYPE;
    if (!aligned(X, 16) || ldx % 8 != 0 || !aligned(codes, 16) || !aligned(scales, 16) || !aligned(Y, y_dtype == ITQ3S_F16 ? 2 : 4) ||
        (status_flags && !aligned(status_flags, 4)))
        return ITQ3S_ERR_ALIGN;
    return itq3s::launch_gemm_weight_side(codes, scales, nullptr, N, K, static_cast<const _Float16*>(X), ldx, M, Y, y_dtype == ITQ3S_F16, ldy, status_flags,
                                          static_cast<hipStream_t>(stream));
}

// ---- measurement aids (include/itq3s_bench.h): the same calls with a pair of events armed for the
// contraction kernel's dispatch, then a wait


int itq3s_matmul_weight_side_timed(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, const void* X, int64_t M, int64_t ldx,
                                   void* Y, int y_dtype, int64_t ldy, uint32_t* status_flags, void* stream, float* kernel_ms) {
    return timed(kernel_ms, [&] { return itq3s_matmul_weight_side(codes, scales, N, K, X, M, ldx, Y, y_dtype, ldy, status_flags, stream); });
}

int itq3s_matmul_grouped_timed(const itq3s_weight* w, int count, int64_t K, const void* X, int64_t M, int64_t ldx, int y_dtype,
                               void* workspace, size_t workspace_bytes, uint32_t* status_flags, void* stream, float* kernel_ms) {
    return timed(kernel_ms, [&] { return itq3s_matmul_grouped(w, count, K, X, M, ldx, y_dtype, workspace, workspace_bytes, status_flags, stream); });
}

int itq3s_matmul_timed(const uint32_t* codes, const uint32_t* scales, int64_t N, int64_t K, const void* X, int64_t M, int64_t ldx,
                       void* Y, int y_dtype, int64_t ldy, void* workspace, size_t workspace_bytes, uint32_t* status_flags, void* stream,
                       float* kernel_ms) {
    if (!codes || !scales || !X || !Y) return ITQ3S_ERR_NULL;
    if (N <= 0 || K <= 0 || M <= 0 || K % 256 != 0 || ldx < K || ldy < N) return ITQ3S_ERR_SHAPE;
    const itq3s_weight w = {codes, scales, N, Y, ldy};
    return itq3s_matmul_grouped_timed(&w, 1, K, X, M, ldx, y_dtype, workspace, workspace_bytes, status_flags, stream, kernel_ms);
}

const char* itq3s_strerror(int status) {
    switch (status) {
        case ITQ3S_OK: return "ok";
        case ITQ3S_ERR_NULL: return "a required pointer is NULL";
        case ITQ3S_ERR_SHAPE: return "bad shape: sizes must be positive, K a multiple of 256, leading dimensions large enough";
        case ITQ3S_ERR_ALIGN: return "pointer or leading dimension not aligned as required";
        case ITQ3S_ERR_DTYPE: return "dtype must be ITQ3S_F32 or ITQ3S_F16";
        case ITQ3S_ERR_WORKSPACE: return "workspace missing or smaller than itq3s_matmul_workspace_bytes()";
        case ITQ3S_ERR_LAUNCH: return "HIP refused the kernel launch";
    }
    return "unknown status";
}

int itq3s_version(void) { return 100; }

}  // extern "C"
