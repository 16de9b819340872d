// Which pixels a posed body can touch, as a bound that errs outwards: the arithmetic of the render kernel's key windows,
// in a header of its own so that a CPU test can compare it with the projected vertices themselves.
//
// Posed template points have view-space coordinates t_i + sum_c M_ic shape_c u_c + M_i2 shape_3 s with |u_c| <= bound_c,
// |u| <= bound_3 and |s| <= 1, so they lie within t_i +- e_i, e_i = the smaller of sum_c |M_ic shape_c| bound_c and
// bound_3 |(M_ic shape_c)_c|, plus |M_i2 shape_3|.  (M is whatever the pose's quaternion makes of it, unit or not.)
// Rounding, here (hardware reciprocals and square roots: 1 ulp) and where the vertices are computed, is below 2^-20 of the
// terms' magnitudes: e_i is widened by 2^-18 of them.  If the box lies in front of the near plane as a whole, its
// projection lies between the extremes of x / z over it; one pixel is added on each side for the projection's own
// rounding (2^-20 of at most 512 pixels) and for the distance from a coordinate to the next pixel centre.  In every other
// case - the box reaches the near plane, something is not a number, or a depth is beyond the range in which the hardware's
// reciprocal is known to be good (beyond 2^126 it returns 0, and half the box would project to the frame's centre) - every
// pixel counts; a box behind the plane as a whole shows nothing.
#ifndef PXR_REACH_H
#define PXR_REACH_H

#include <cstdint>

#ifdef __HIPCC__
#define PXR_BOTH __host__ __device__ __forceinline__
#else
#define PXR_BOTH inline
#endif

namespace pxr {

constexpr float kReachDepthMin = 0x1p-100f, kReachDepthMax = 0x1p100f;

// e_i of one axis: m = its row of M, t = its coordinate of the origin.  `root` = square root, 1 ulp.
template <class Root>
PXR_BOTH float half_extent(float m0, float m1, float m2, float t, float shape0, float shape1, float shape2, float shape3,
                           float bound0, float bound1, float bound2, float bound3, Root root) {
    const float p = __builtin_fabsf(m0 * shape0), q = __builtin_fabsf(m1 * shape1), r = __builtin_fabsf(__builtin_fabsf(m2) * shape2);
    const float sum = p * bound0 + q * bound1 + r * bound2;
    const float ball = bound3 * root(p * p + q * q + r * r);
    float e = ball >= 0x1p-40f && ball < sum ? ball : sum;  // (tiny squares may vanish: not below 2^-40)
    e += __builtin_fabsf(__builtin_fabsf(m2) * shape3);
    return e + 0x1p-18f * (e + sum + __builtin_fabsf(t));
}

struct AxisReach {
    uint32_t begin, end;  // pixels [begin, end) of the axis; none if begin >= end
    PXR_BOTH bool none() const { return begin >= end; }
};

// An axis of the image, n pixels long, that points along view coordinates [lo, hi] of a box with depths [z_lo, z_hi]:
// projected as focal * x / z + half.  (near_inv and far_inv: the depths' reciprocals.)
PXR_BOTH AxisReach axis_reach(float lo, float hi, float z_lo, float z_hi, float near_inv, float far_inv, float focal, float half,
                              uint32_t n, float z_near) {
    const float first = __builtin_fmaf(focal, lo * (lo > 0.0f ? far_inv : near_inv), half);
    const float last = __builtin_fmaf(focal, hi * (hi > 0.0f ? near_inv : far_inv), half);
    AxisReach a = {0u, n};
    if (z_lo > z_near && z_lo >= kReachDepthMin && z_hi <= kReachDepthMax && first <= last) {  // (no NaN gets here)
        a.begin = (uint32_t)__builtin_fminf(__builtin_fmaxf(first - 1.0f, 0.0f), 512.0f);
        const uint32_t end = (uint32_t)__builtin_fminf(__builtin_fmaxf(last + 2.0f, 0.0f), 512.0f);
        a.end = end < n ? end : n;
    }
    if (z_hi < z_near) a.end = 0u;
    return a;
}

}  // namespace pxr

#endif
