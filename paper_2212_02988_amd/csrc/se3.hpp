// Rotations and pose increments in double precision (device side): skew
// matrices, SO(3) exponential (with its left Jacobian) and logarithm,
// quaternion <-> matrix, the pose error e = (t_a - t_b, Log(R_a R_b^T)) and
// the left, world-frame retraction t <- t + d_t, R <- Exp(d_theta) R.
#pragma once
#include "common.hpp"

namespace prism {

__device__ inline void skew(const double v[3], double K[9]) {
    K[0] = 0.0;   K[1] = -v[2]; K[2] = v[1];
    K[3] = v[2];  K[4] = 0.0;   K[5] = -v[0];
    K[6] = -v[1]; K[7] = v[0];  K[8] = 0.0;
}

__device__ inline void mat3mul(const double A[9], const double B[9], double C[9]) {
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) C[i * 3 + j] = A[i * 3] * B[j] + A[i * 3 + 1] * B[3 + j] + A[i * 3 + 2] * B[6 + j];
}

// 1/sqrt(x) and sqrt(x) of a positive normal number: the hardware estimate
// (about 2^-23) and two steps of Goldschmidt's coupled Newton iteration, to
// within an ulp or two.  The pose algebra runs on one lane's dependent chain,
// where a square root and a division cost about 300 clocks and this about 100.
__device__ __forceinline__ double rsqrt64(double x, double* root = nullptr) {
    double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = __builtin_fma(-h, g, 0.5);
        g = __builtin_fma(g, r, g);
        h = __builtin_fma(h, r, h);
    }
    if (root) *root = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return 2.0 * h;
}

// Coefficients of Exp and its left Jacobian at angle th: A = sin(th)/th,
// B = (1 - cos(th))/th^2, C = (th - sin(th))/th^3, in powers of th^2: eight
// terms are exact in double precision to th = 1/2 (and keep the digits that
// the differences lose); the functions of a larger angle stay out of the
// callers' straight-line code.
struct ExpCoef {
    double A, B, C;
};
static __device__ __attribute__((noinline)) ExpCoef exp_coef_far(double th2) {
    const double th = sqrt(th2), s = sin(th);
    return ExpCoef{s / th, (1.0 - cos(th)) / th2, (th - s) / (th2 * th)};
}
__device__ __forceinline__ ExpCoef exp_coef(double th2) {
    ExpCoef o{0.0, 0.0, 0.0};
    // 1/(2n+1)!, 1/(2n+2)!, 1/(2n+3)! with alternating signs, n = 7 .. 0
    constexpr double f[18] = {1.0, 1.0, 2.0, 6.0, 24.0, 120.0, 720.0, 5040.0, 40320.0, 362880.0, 3628800.0, 39916800.0,
                              479001600.0, 6227020800.0, 87178291200.0, 1307674368000.0, 20922789888000.0,
                              355687428096000.0};
#pragma unroll
    for (int n = 7; n >= 0; --n) {
        const double sg = n & 1 ? -1.0 : 1.0;
        o.A = __builtin_fma(th2, o.A, sg / f[2 * n + 1]);
        o.B = __builtin_fma(th2, o.B, sg / f[2 * n + 2]);
        o.C = __builtin_fma(th2, o.C, sg / f[2 * n + 3]);
    }
    if (th2 > 0.25) o = exp_coef_far(th2);
    return o;
}

// Exp(phi) (Rodrigues) and the left Jacobian J_l(phi)
__device__ inline void so3_exp(const double phi[3], double R[9], double* Jl) {
    const ExpCoef f = exp_coef(phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2]);
    double K[9], K2[9];
    skew(phi, K);
    mat3mul(K, K, K2);
    for (int e = 0; e < 9; ++e) {
        double I = (e % 4 == 0) ? 1.0 : 0.0;
        R[e] = I + f.A * K[e] + f.B * K2[e];
        if (Jl) Jl[e] = I + f.B * K[e] + f.C * K2[e];
    }
}

// Exp alone, with [w]x^2 = w w^T - th^2 I
__device__ inline void so3_exp_step(const double w[3], double E[9]) {
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    const ExpCoef f = exp_coef(th2);
    const double A = f.A, B = f.B;
    // E = I + A [w]x + B [w]x^2, with [w]x^2 = w w^T - th2 I
    const double Bw[3] = {B * w[0], B * w[1], B * w[2]};
    const double d = 1.0 - B * th2;
    E[0] = __builtin_fma(Bw[0], w[0], d);
    E[4] = __builtin_fma(Bw[1], w[1], d);
    E[8] = __builtin_fma(Bw[2], w[2], d);
    const double xy = Bw[0] * w[1], xz = Bw[0] * w[2], yz = Bw[1] * w[2];
    E[1] = __builtin_fma(-A, w[2], xy);
    E[3] = __builtin_fma(A, w[2], xy);
    E[2] = __builtin_fma(A, w[1], xz);
    E[6] = __builtin_fma(-A, w[1], xz);
    E[5] = __builtin_fma(-A, w[0], yz);
    E[7] = __builtin_fma(A, w[0], yz);
}

struct Vec3 {
    double x, y, z;
};
struct Mat9 {
    double m[9];
};
// rotation vector of angles beyond the series below
static __device__ __attribute__((noinline)) Vec3 so3_log_far(Mat9 M) {
    const double* R = M.m;
    double c = (R[0] + R[4] + R[8] - 1.0) * 0.5;
    c = fmin(1.0, fmax(-1.0, c));
    double th = acos(c);
    double v[3] = {R[7] - R[5], R[2] - R[6], R[3] - R[1]};
    if (M_PI - th < 1e-6) {
        // near pi: axis from the column of (R + I)/2 with the largest diagonal
        double ax0, ax1, ax2;
        if (R[0] >= R[4] && R[0] >= R[8]) {
            ax0 = (R[0] + 1.0) * 0.5; ax1 = R[3] * 0.5; ax2 = R[6] * 0.5;
        } else if (R[4] >= R[8]) {
            ax0 = R[1] * 0.5; ax1 = (R[4] + 1.0) * 0.5; ax2 = R[7] * 0.5;
        } else {
            ax0 = R[2] * 0.5; ax1 = R[5] * 0.5; ax2 = (R[8] + 1.0) * 0.5;
        }
        double n = sqrt(ax0 * ax0 + ax1 * ax1 + ax2 * ax2);
        return Vec3{th * ax0 / n, th * ax1 / n, th * ax2 / n};
    }
    double f = th / (2.0 * sin(th));
    return Vec3{f * v[0], f * v[1], f * v[2]};
}

// Log: th / sin(th) = asin(s) / s in powers of s^2 = sin(th)^2 while s < 0.1
// (ten terms are exact in double precision there; an arc cosine loses digits
// at small angles and takes about 300 clocks)
__device__ inline void so3_log(const double R[9], double w[3]) {
    const double v[3] = {R[7] - R[5], R[2] - R[6], R[3] - R[1]};
    const double s2 = 0.25 * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    if (s2 < 0.01 && R[0] + R[4] + R[8] > 1.0) {
        // (2n)! / (4^n n!^2 (2n + 1))
        constexpr double k[10] = {1.0, 1.0 / 6.0, 3.0 / 40.0, 5.0 / 112.0, 35.0 / 1152.0, 63.0 / 2816.0,
                                  231.0 / 13312.0, 143.0 / 10240.0, 6435.0 / 557056.0, 12155.0 / 1245184.0};
        double f = k[9];
#pragma unroll
        for (int n = 8; n >= 0; --n) f = __builtin_fma(s2, f, k[n]);
        for (int i = 0; i < 3; ++i) w[i] = 0.5 * f * v[i];
        return;
    }
    Mat9 M;
    for (int i = 0; i < 9; ++i) M.m[i] = R[i];
    const Vec3 o = so3_log_far(M);
    w[0] = o.x;
    w[1] = o.y;
    w[2] = o.z;
}

// unit-quaternion rotation for the pose algebra (one reciprocal)
__device__ inline void quat_to_R9(const double q[4], double R[9]) {
    double in = rsqrt64(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    double w = q[0] * in, x = q[1] * in, y = q[2] * in, z = q[3] * in;
    R[0] = 1.0 - 2.0 * (y * y + z * z);
    R[1] = 2.0 * (x * y - w * z);
    R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);
    R[4] = 1.0 - 2.0 * (x * x + z * z);
    R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);
    R[7] = 2.0 * (y * z + w * x);
    R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// rotation matrix -> unit quaternion (w >= 0), branch on the largest of
// trace and diagonal (constant indices only, so nothing leaves registers)
__device__ inline void R9_to_quat(const double R[9], double q[4]) {
    double tr = R[0] + R[4] + R[8];
    if (tr > 0.0) {
        double s, is = 0.5 * rsqrt64(tr + 1.0, &s);
        s *= 2.0;
        q[0] = 0.25 * s;
        q[1] = (R[7] - R[5]) * is;
        q[2] = (R[2] - R[6]) * is;
        q[3] = (R[3] - R[1]) * is;
    } else if (R[0] >= R[4] && R[0] >= R[8]) {
        double s, is = 0.5 * rsqrt64(1.0 + R[0] - R[4] - R[8], &s);
        s *= 2.0;
        q[0] = (R[7] - R[5]) * is;
        q[1] = 0.25 * s;
        q[2] = (R[1] + R[3]) * is;
        q[3] = (R[2] + R[6]) * is;
    } else if (R[4] >= R[8]) {
        double s, is = 0.5 * rsqrt64(1.0 + R[4] - R[8] - R[0], &s);
        s *= 2.0;
        q[0] = (R[2] - R[6]) * is;
        q[1] = (R[1] + R[3]) * is;
        q[2] = 0.25 * s;
        q[3] = (R[5] + R[7]) * is;
    } else {
        double s, is = 0.5 * rsqrt64(1.0 + R[8] - R[0] - R[4], &s);
        s *= 2.0;
        q[0] = (R[3] - R[1]) * is;
        q[1] = (R[2] + R[6]) * is;
        q[2] = (R[5] + R[7]) * is;
        q[3] = 0.25 * s;
    }
    if (q[0] < 0.0) {
        q[0] = -q[0]; q[1] = -q[1]; q[2] = -q[2]; q[3] = -q[3];
    }
    double in = rsqrt64(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    q[0] *= in; q[1] *= in; q[2] *= in; q[3] *= in;
}

// tangent of pose a relative to pose b: (t_a - t_b, Log(R_a R_b^T))
__device__ inline void pose_err(const prism_pose& a, const prism_pose& b, double e[6]) {
    double Ra[9], Rb[9], M[9];
    quat_to_R9(a.q, Ra);
    quat_to_R9(b.q, Rb);
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            M[i * 3 + j] = Ra[i * 3] * Rb[j * 3] + Ra[i * 3 + 1] * Rb[j * 3 + 1] + Ra[i * 3 + 2] * Rb[j * 3 + 2];
    for (int i = 0; i < 3; ++i) e[i] = a.t[i] - b.t[i];
    so3_log(M, e + 3);
}

// t <- t + dt, R <- Exp(dtheta) R
__device__ inline void retract(prism_pose& p, const double d[6]) {
    double E[9], R[9], R2[9];
    so3_exp(d + 3, E, nullptr);
    quat_to_R9(p.q, R);
    mat3mul(E, R, R2);
    for (int i = 0; i < 3; ++i) p.t[i] += d[i];
    R9_to_quat(R2, p.q);
}

}  // namespace prism
