// The fp32 function of the general propagation's fills: the logarithm of an edge's term.
#ifndef SPP_FP32_H
#define SPP_FP32_H

namespace spp {

// log1p(-x) for 0 < x <= 1 to 2.4 fp32 ulp (against 64 bits, whatever the reciprocal's last place).  All terms of a vertex's sum have one sign, so the
// sum's relative error is at most the largest of its terms'; the library's fp32 and fp64 routines
// carry extended precision that is of no use here and were 90 and 117 of the walk's instructions per
// edge.  Below 1/4 the atanh series in s = x / (2 - x) <= 1/7 (six terms: the next is below 2^-33
// of the first); above, the logarithm of 1 - x, whose rounding error is at most 2^-25 against a
// result of at least 0.28.
__device__ __forceinline__ float bin_log1p_neg(float x) {
    // x / (2 - x) from the reciprocal's estimate and one correction: to half a unit as the division, four instructions
    // instead of eleven (2 - x lies in [1, 2])
    const float d = 2.0f - x, r = __builtin_amdgcn_rcpf(d), s0 = x * r;
    const float s = __fmaf_rn(__fmaf_rn(-s0, d, x), r, s0);
    const float z = s * s;
    float q = 1.0f / 11.0f;
    q = __fmaf_rn(q, z, 1.0f / 9.0f);
    q = __fmaf_rn(q, z, 1.0f / 7.0f);
    q = __fmaf_rn(q, z, 1.0f / 5.0f);
    q = __fmaf_rn(q, z, 1.0f / 3.0f);
    q = __fmaf_rn(q, z, 1.0f);
    const float small = __fmaf_rn(-2.0f * s, q, 0.0f);     // +0 for x = 0
    const float large = __logf(1.0f - x);
    return x < 0.25f ? small : large;
}

}  // namespace spp
#endif
