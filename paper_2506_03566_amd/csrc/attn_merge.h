// The merge of a row's attention splits, shared by attn_merge_kernel and by the output projection that merges for itself: the
// same operations in the same order, so a row gets the same bits from either.
#pragma once
#include "device_utils.h"

namespace poss {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Four columns of one (row, head): partial outputs o[s * stride * dh ..] and (maximum, sum) pairs ml[s * stride * 2 ..] of n_splits
// <= NR splits; slots beyond n_splits re-read the last split and are not used.  load() only requests.
template <int NR>
struct MergeQuad {
    float ms[NR], ls[NR];
    f32x4 v[NR];
    __device__ __forceinline__ void load(const float *o, const float *ml, size_t stride, int dh, int n_splits) {
#pragma unroll
        for (int s = 0; s < NR; ++s) {
            const int sc = s < n_splits ? s : n_splits - 1;
            const float2 x = *reinterpret_cast<const float2 *>(ml + (size_t)sc * stride * 2);
            ms[s] = x.x; ls[s] = x.y;
            v[s] = *reinterpret_cast<const f32x4 *>(o + (size_t)sc * stride * dh);
        }
    }
    // num / den is the row's output.  A split without visible keys has weight 0 and O = 0; maxima are in the log2 domain.
    __device__ __forceinline__ void merge(int n_splits, f32x4 &num, float &den) const {
        float M = -INFINITY;
        den = 0.f;
        num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NR; ++s) if (s < n_splits) M = fmaxf(M, ms[s]);
#pragma unroll
        for (int s = 0; s < NR; ++s)
            if (s < n_splits) {
                const float w = ms[s] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms[s] - M);
                den += w * ls[s];
                num += w * v[s];
            }
    }
};

}  // namespace poss
