// Shared by the streaming kernels (itq3s_gemv.hip, itq3s_rows.hip): the tensor list of a launch and the
// pieces of the packed operand.
#pragma once
#include "itq3s_dev.h"
#include "itq3s_kernels.h"

namespace itq3s {

constexpr int kRawBuffer = 0x00027000;  // buffer descriptor word 3: raw buffer of 32-bit elements
constexpr int kLoadNT = 2;              // cache policy of the weight loads: nontemporal (read once)

// One launch serves up to kGemvMaxGroup weight tensors that share K and the activations (the
// projections of one layer that read the same input).  Their 16-row tiles are numbered as one list,
// tensor after tensor, and split evenly over the workgroups; a workgroup's tiles may belong to two
// tensors.
struct GemvTensor {
    const uint32_t* codes;
    const uint32_t* scales;
    const uint32_t* subscales;  // the 116-byte variant's sub-scale array, or null
    void* Y;
    int64_t N, ldy;
    int v_begin;  // position of this tensor's first row tile in the list (0x7fffffff for unused entries)
    int pad_;
};

__device__ __forceinline__ half8 as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    u32x4 u = {a, b, c, d};
    return __builtin_bit_cast(half8, u);
}

// Fills the tensor list of a launch; returns the number of row tiles, or -1.
inline int64_t fill_tensors(GemvTensor (&list)[kGemvMaxGroup], const GemvWeight* w, int count) {
    int64_t nt_total = 0;
    for (int i = 0; i < kGemvMaxGroup; ++i) {
        GemvTensor& t = list[i];
        if (i < count) {
            t.codes = w[i].codes; t.scales = w[i].scales; t.subscales = w[i].subscales; t.Y = w[i].Y; t.N = w[i].N; t.ldy = w[i].ldy;
            if (t.subscales != nullptr && count != 1) return -1;
            if (nt_total > 0x7fffffff) return -1;
            t.v_begin = (int)nt_total;
            nt_total += (w[i].N + 15) / 16;
        } else {
            t = list[0];
            t.v_begin = 0x7fffffff;
        }
        t.pad_ = 0;
    }
    return nt_total < 0x7fffffff ? nt_total : -1;
}

}  // namespace itq3s
