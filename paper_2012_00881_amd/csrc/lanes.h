// Sums over the 2 or 4 neighbouring lanes that share a cell (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace wq {

// The value of the quad's lane q ^ X (X = 1 or 2), by DPP.
template <int X>
__device__ __forceinline__ double quad_xor(double v) {
    constexpr int ctrl = X == 1 ? 0xB1 : 0x4E;  // quad_perm [1, 0, 3, 2], [2, 3, 0, 1]
    const unsigned long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Joins the corner values s[4] of a cell's LANES lanes in a fixed order; lane q
// puts the corners that it ends with at out[corner * stride].
template <int LANES>
__device__ __forceinline__ void join_corners(double s0, double s1, double s2, double s3, int q, double* out,
                                             int stride) {
    static_assert(LANES == 2 || LANES == 4, "lanes per cell");
    const bool b0 = q & 1, b1 = q & 2;
    const double lo = (b0 ? s1 : s0) + quad_xor<1>(b0 ? s0 : s1);  // corner b0 of lanes q, q ^ 1
    const double hi = (b0 ? s3 : s2) + quad_xor<1>(b0 ? s2 : s3);  // corner 2 + b0
    if constexpr (LANES == 2) {
        out[q * stride] = lo;
        out[(2 + q) * stride] = hi;
    } else {
        out[q * stride] = (b1 ? hi : lo) + quad_xor<2>(b1 ? lo : hi);
    }
}

}  // namespace wq
