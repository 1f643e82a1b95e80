// Shared by the kernels that index the pixels of a batch as one flat range (conv_gemm_f32.hip,
// conv_wgrad_gemm_f32.hip).
#pragma once

#include "kernels.h"

namespace rvn {
namespace flat {

// Multiplier for div_u by d.
inline uint32_t magic(int d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d); }

// e / d for 0 <= e < 2^31 with m = magic(d): the estimate is exact or one short.
__device__ __forceinline__ int div_u(int e, int d, uint32_t m) {
    if (m == 0) return e;
    int q = (int)__umulhi((uint32_t)e, m);
    return e - q * d >= d ? q + 1 : q;
}

// Element offsets are 32-bit byte offsets: whether they reach all of a tensor of c channels.
constexpr int64_t kMaxElems = (int64_t)1 << 30;
inline bool fits(const View &v, int c, const Geo &g) {
    return (int64_t)g.n * v.sn + (int64_t)c * v.sc + (int64_t)g.h * g.w < kMaxElems;
}

}  // namespace flat
}  // namespace rvn
