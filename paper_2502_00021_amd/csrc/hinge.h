// The arithmetic of a hinge: the pose of a body from its parent's and its joint angle.  Shared by the kinematics kernel
// (a lane per frame) and the render kernel's own kinematics stage (a lane per body).
//
// Arithmetic: fp32, explicit fmaf, no contraction.  sin and cos of half the
// hinge angle come from a two-constant Cody-Waite reduction by pi/2 and two
// Taylor polynomials (within 1.25 * 2^-24 of the true values for hinge angles
// up to +-65536 rad); an angle beyond that, or a non-finite one, gives NaN for
// both, so the body and its descendants drop out of the frame.
#ifndef PXR_HINGE_H
#define PXR_HINGE_H

#include <hip/hip_runtime.h>

#include "pxr_internal.h"

namespace pxr {

constexpr float kMaxHingeAngle = 65536.0f;  // radians; the reduction below is accurate up to here

__device__ __forceinline__ void sincos_half(float theta, float& s, float& c) {
    const float h = 0.5f * theta;
    const float kf = __builtin_rintf(h * 0.636619772f);  // nearest multiple of pi/2, ties to even
    float r = __builtin_fmaf(kf, -1.57079625f, h);
    r = __builtin_fmaf(kf, -7.54978942e-08f, r);
    const float r2 = r * r;
    float ps = __builtin_fmaf(r2, 2.75573192e-06f, -1.98412698e-04f);
    ps = __builtin_fmaf(ps, r2, 8.33333333e-03f);
    ps = __builtin_fmaf(ps, r2, -1.66666667e-01f);
    const float sp = __builtin_fmaf(r * r2, ps, r);
    float pc = __builtin_fmaf(r2, -2.75573192e-07f, 2.48015873e-05f);
    pc = __builtin_fmaf(pc, r2, -1.38888889e-03f);
    pc = __builtin_fmaf(pc, r2, 4.16666667e-02f);
    pc = __builtin_fmaf(pc, r2, -0.5f);
    const float cp = __builtin_fmaf(pc, r2, 1.0f);
    const int q = (int)kf & 3;  // (|kf| < 2^15 inside the domain)
    s = q == 0 ? sp : (q == 1 ? cp : (q == 2 ? -sp : -cp));
    c = q == 0 ? cp : (q == 1 ? -sp : (q == 2 ? -cp : sp));
    if (!(__builtin_fabsf(theta) <= kMaxHingeAngle)) s = c = __builtin_nanf("");
}

// Row r of the rotation matrix of quaternion (w,x,y,z) applied to v, as
// fma(m0, v0, fma(m1, v1, m2 * v2)); same matrix formulas as the renderer's
// vertex stage.
__device__ __forceinline__ void rotate(float w, float x, float y, float z, float v0, float v1, float v2, float out[3]) {
    const float m00 = 1.0f - 2.0f * (y * y + z * z), m01 = 2.0f * (x * y - w * z), m02 = 2.0f * (x * z + w * y);
    const float m10 = 2.0f * (x * y + w * z), m11 = 1.0f - 2.0f * (x * x + z * z), m12 = 2.0f * (y * z - w * x);
    const float m20 = 2.0f * (x * z - w * y), m21 = 2.0f * (y * z + w * x), m22 = 1.0f - 2.0f * (x * x + y * y);
    out[0] = __builtin_fmaf(m00, v0, __builtin_fmaf(m01, v1, m02 * v2));
    out[1] = __builtin_fmaf(m10, v0, __builtin_fmaf(m11, v1, m12 * v2));
    out[2] = __builtin_fmaf(m20, v0, __builtin_fmaf(m21, v1, m22 * v2));
}

// Pose (position, quaternion) of a hinged body from its parent's and the cosine and sine of its half angle.
__device__ __forceinline__ void hinge_pose(const SkeletonRecord& t, const float pp[7], float cs, float sn, float o[7]) {
    const float ppx = pp[0], ppy = pp[1], ppz = pp[2], pw = pp[3], px = pp[4], py = pp[5], pz = pp[6];
    const float jw = cs, jx = sn * t.axis[0], jy = sn * t.axis[1], jz = sn * t.axis[2];
    // body orientation = parent orientation (x) hinge rotation (Hamilton product)
    const float qw = __builtin_fmaf(-pz, jz, __builtin_fmaf(-py, jy, __builtin_fmaf(-px, jx, pw * jw)));
    const float qx = __builtin_fmaf(py, jz, __builtin_fmaf(-pz, jy, __builtin_fmaf(px, jw, pw * jx)));
    const float qy = __builtin_fmaf(pz, jx, __builtin_fmaf(-px, jz, __builtin_fmaf(py, jw, pw * jy)));
    const float qz = __builtin_fmaf(px, jy, __builtin_fmaf(-py, jx, __builtin_fmaf(pz, jw, pw * jz)));
    float t1[3], t2[3];
    rotate(pw, px, py, pz, t.anchor[0], t.anchor[1], t.anchor[2], t1);  // hinge position, parent frame -> world
    rotate(qw, qx, qy, qz, t.offset[0], t.offset[1], t.offset[2], t2);  // body centre relative to the hinge
    o[0] = (ppx + t1[0]) + t2[0];
    o[1] = (ppy + t1[1]) + t2[1];
    o[2] = (ppz + t1[2]) + t2[2];
    o[3] = qw;
    o[4] = qx;
    o[5] = qy;
    o[6] = qz;
}

}  // namespace pxr

#endif
