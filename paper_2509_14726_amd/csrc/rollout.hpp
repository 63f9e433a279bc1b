// Quadrotor dynamics (Sec. III-A, Eq. (2)): the parts that the rollouts share.
//
// State x = [p, v, q = (w, x, y, z), omega]; input = four rotor thrusts held
// over the step.  The quaternion is scaled back to unit norm after every
// step.  Binary32 rollouts carry the state in plain binary32: over horizons
// of up to 256 steps their cost errors stay near 1e-6 of the cost scale (the
// magnitudes of the terms), and the cost sums themselves are compensated.
#pragma once

#include "device.hpp"

namespace mppi {

template <typename Real> struct Model {
    Real inv_m, g, arm_s, c_tau;
    Real ijx, ijy, ijz, gx, gy, gz;
    Real d0, d1, d2;
    bool drag;

    __device__ __forceinline__ explicit Model(const KArgs &a)
        : inv_m((Real)a.inv_mass), g((Real)a.gravity), arm_s((Real)a.arm_s), c_tau((Real)a.c_tau),
          ijx((Real)a.inv_J[0]), ijy((Real)a.inv_J[1]), ijz((Real)a.inv_J[2]),
          gx((Real)a.gyro[0]), gy((Real)a.gyro[1]), gz((Real)a.gyro[2]),
          d0((Real)a.drag[0]), d1((Real)a.drag[1]), d2((Real)a.drag[2]), drag(a.has_drag != 0) {}
};

// Per-step input terms: collective thrust over mass and torque over inertia.
template <typename Real> struct StepInput {
    Real fm, tx, ty, tz;
};

template <typename Real>
__device__ __forceinline__ StepInput<Real> step_input(const Model<Real> &M, Real u0, Real u1, Real u2,
                                                       Real u3)
{
    StepInput<Real> s;
    s.fm = ((u0 + u1) + (u2 + u3)) * M.inv_m;
    s.tx = M.arm_s * ((u0 + u1) - (u2 + u3)) * M.ijx;
    s.ty = M.arm_s * ((u1 + u2) - (u0 + u3)) * M.ijy;
    s.tz = M.c_tau * ((u0 + u2) - (u1 + u3)) * M.ijz;
    return s;
}

// Acceleration of one RK4 stage: F/m times the thrust direction (third column
// of R(q); the factor 2 of its first two components rides on F/m, exact: a
// power of two), gravity and the rotor drag - R D R^T v.
template <bool DRAG, typename Real>
__device__ __forceinline__ void stage_accel(const Model<Real> &M, Real fm, const Real *q, const Real *v, Real *kv)
{
    const Real fm2 = Real(2) * fm;
    const Real r3z = Real(1) - Real(2) * (q[1] * q[1] + q[2] * q[2]);
    kv[0] = fm2 * (q[1] * q[3] + q[0] * q[2]);
    kv[1] = fm2 * (q[2] * q[3] - q[0] * q[1]);
    kv[2] = fm * r3z - M.g;
    if (DRAG) {
        const Real qw = q[0], qx = q[1], qy = q[2], qz = q[3];
        const Real r3x = Real(2) * (q[1] * q[3] + q[0] * q[2]);
        const Real r3y = Real(2) * (q[2] * q[3] - q[0] * q[1]);
        const Real r11 = Real(1) - Real(2) * (qy * qy + qz * qz), r12 = Real(2) * (qx * qy - qw * qz);
        const Real r21 = Real(2) * (qx * qy + qw * qz), r22 = Real(1) - Real(2) * (qx * qx + qz * qz);
        const Real r31 = Real(2) * (qx * qz - qw * qy), r32 = Real(2) * (qy * qz + qw * qx);
        const Real b0 = M.d0 * (r11 * v[0] + r21 * v[1] + r31 * v[2]);
        const Real b1 = M.d1 * (r12 * v[0] + r22 * v[1] + r32 * v[2]);
        const Real b2 = M.d2 * (r3x * v[0] + r3y * v[1] + r3z * v[2]);
        kv[0] -= r11 * b0 + r12 * b1 + r3x * b2;
        kv[1] -= r21 * b0 + r22 * b1 + r3y * b2;
        kv[2] -= r31 * b0 + r32 * b1 + r3z * b2;
    }
}

// Scale a quaternion back to unit norm: the hardware reciprocal square root,
// which is all binary32 needs; binary64 refines it (about 2^-24) in one
// third-order step from the exactly formed residual.  Against a square root
// and four divisions, each correctly rounded, the binary64 attitude step issues
// some 70 instructions fewer; errors against extended precision over 4e6 draws
// near unit norm, in half ulps: mean 0.511, max 2.00 -> 0.491, 1.99.
__device__ __forceinline__ void renormalize(float *q)
{
    const float r = inv_sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] *= r;
}
__device__ __forceinline__ void renormalize(double *q)
{
    const double n2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3];
    const double y = __builtin_amdgcn_rsq(n2);
    const double t = n2 * y, tl = __builtin_fma(n2, y, -t);
    const double e = __builtin_fma(-tl, y, __builtin_fma(-t, y, 1.0));
    const double r = __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] *= r;
}

}  // namespace mppi
