// Visual-inertial factors on the GPU (Background Eq. 8; Sec. V-C): IMU
// preintegration between consecutive keyframes, the inertial residual with
// first-order bias correction, and rectified stereo reprojection.  Residuals
// are written once over a generic scalar; their Jacobians come from forward-
// mode automatic differentiation (Sec. IV-C), one lane per (factor, column)
// with the column's local perturbation seeded.  Keyframe state: rotation
// R (world <- body, passed as an angle-axis vector), position p, velocity v,
// gyroscope bias b_g, accelerometer bias b_a; Jacobian columns are the right
// perturbation R Exp(dtheta) and additive p, v, b.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <vector>

#include "gba.h"
#include "gba_autodiff.h"
#include "gba_device.h"
#include "gba_vi_bufs.h"
#include "gba_vi_order.h"
#include "gba_vi_rule.h"

namespace gba {
namespace vi {

constexpr double kSmall = 1e-8;   // |phi|^2 below which Exp / Log use their series
constexpr double kGravity[3] = {0.0, 0.0, -9.81};

// layout of one preintegrated interval (doubles)
enum {
    kDt = 0, kDR = 1, kDV = 10, kDP = 13, kJRg = 16, kJvg = 25, kJva = 34, kJpg = 43, kJpa = 52,
    kBg0 = 61, kBa0 = 64, kCov = 67, kPreStride = 148
};

template <typename S>
__device__ __forceinline__ void skew(const S (&v)[3], S (&K)[3][3]) {
    const S z = v[0] * 0.0;
    K[0][0] = z;     K[0][1] = -v[2]; K[0][2] = v[1];
    K[1][0] = v[2];  K[1][1] = z;     K[1][2] = -v[0];
    K[2][0] = -v[1]; K[2][1] = v[0];  K[2][2] = z;
}

template <typename A, typename B, typename C>
__device__ __forceinline__ void mm(const A (&a)[3][3], const B (&b)[3][3], C (&c)[3][3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) c[r][k] = a[r][0] * b[0][k] + a[r][1] * b[1][k] + a[r][2] * b[2][k];
}

template <typename A, typename B, typename C>
__device__ __forceinline__ void mtm(const A (&a)[3][3], const B (&b)[3][3], C (&c)[3][3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) c[r][k] = a[0][r] * b[0][k] + a[1][r] * b[1][k] + a[2][r] * b[2][k];
}

// Exp of a 3-vector: I + a K + b K^2, a = sin t / t, b = (1 - cos t) / t^2
// (series below |phi|^2 = kSmall); generic over double and Dual<double>.
template <typename S>
__device__ __forceinline__ void so3_exp(const S (&phi)[3], S (&R)[3][3]) {
    const S t2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
    S a, b;
    if (ad_value(t2) < kSmall) {
        a = 1.0 - t2 / 6.0;
        b = 0.5 - t2 / 24.0;
    } else {
        const S t = ad_sqrt(t2);
        a = ad_sin(t) / t;
        b = (1.0 - ad_cos(t)) / t2;
    }
    S K[3][3], K2[3][3];
    skew(phi, K);
    mm(K, K, K2);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) R[r][c] = a * K[r][c] + b * K2[r][c] + (r == c ? 1.0 : 0.0);
}

// Log of a rotation matrix: theta = atan2(|v|, (tr R - 1) / 2) with v the
// axial part; theta / sin theta by its series below |v|^2 = kSmall.
template <typename S>
__device__ __forceinline__ void so3_log(const S (&R)[3][3], S (&phi)[3]) {
    const S c = 0.5 * (R[0][0] + R[1][1] + R[2][2] - 1.0);
    const S v[3] = {0.5 * (R[2][1] - R[1][2]), 0.5 * (R[0][2] - R[2][0]), 0.5 * (R[1][0] - R[0][1])};
    const S s2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    S f;
    if (ad_value(s2) < kSmall) {
        f = 1.0 + s2 / 6.0 + 0.075 * s2 * s2;
    } else {
        const S s = ad_sqrt(s2);
        f = ad_atan2(s, c) / s;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) phi[k] = v[k] * f;
}

__device__ inline void right_jacobian(const double (&phi)[3], double (&J)[3][3]) {
    const double t2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
    double a, b;
    if (t2 < kSmall) {
        a = 0.5;
        b = 1.0 / 6.0;
    } else {
        const double t = sqrt(t2);
        a = (1.0 - cos(t)) / t2;
        b = (t - sin(t)) / (t2 * t);
    }
    double K[3][3], K2[3][3];
    skew(phi, K);
    mm(K, K, K2);
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) J[r][c] = (r == c ? 1.0 : 0.0) - a * K[r][c] + b * K2[r][c];
}

// ---------------------------------------------------------- preintegration
// 16 lanes per interval (a DPP row): the samples [off[f], off[f+1]) with the
// interval's bias estimates; deltas, bias Jacobians and the covariance
// (continuous noise densities sg, sa) are propagated with the values before
// each step.  A sample's Exp and right Jacobian depend on its reading alone:
// 16 samples at a time, one per lane, go to LDS; the chain over the samples
// then has the covariance by columns (lane c < 9), the bias Jacobians by
// columns (lane c < 3) and the rotation in every lane, with the columns
// exchanged inside the row.  Bound by that chain's instructions: 76 us at
// 200 Hz over 0.25 s (1.5 us a sample; 350 us with one lane per interval, most
// of it the dense 9 x 9 products and the trigonometry).
constexpr int kPreSample = 21;   // Exp (9), right Jacobian (9), acceleration (3)
template <int kLane>
__device__ __forceinline__ double row_lane(double v) {   // row_newbcast
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + kLane, 0xF, 0xF, true);
}

__global__ __launch_bounds__(64) void k_preintegrate(int n, const long long* __restrict__ off,
                                                    const double* __restrict__ gyro,
                                                    const double* __restrict__ acc, double dt,
                                                    const double* __restrict__ bias0, double sg,
                                                    double sa, double* __restrict__ out) {
    __shared__ double smp_s[4][16 * kPreSample];
    __shared__ double cov_s[4][81];
    const int grp = (int)threadIdx.x >> 4, c = (int)threadIdx.x & 15, c3 = c % 3;
    const int f = (int)blockIdx.x * 4 + grp;
    const long long s0 = f < n ? off[f] : 0;
    const long long cnt = f < n ? off[f + 1] - s0 : 0;
    double b0[6];
    for (int k = 0; k < 6; ++k) b0[k] = f < n ? bias0[6 * f + k] : 0.0;
    const double qg = sg * sg / dt, qa = sa * sa / dt;
    double dR[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}}, dv[3] = {0, 0, 0}, dp[3] = {0, 0, 0};
    // columns: of the rotation, the bias Jacobians (c < 3), the covariance (c < 9)
    double Rc[3] = {c == 0 ? 1.0 : 0.0, c == 1 ? 1.0 : 0.0, c == 2 ? 1.0 : 0.0};
    double jrg[3] = {}, jvg[3] = {}, jva[3] = {}, jpg[3] = {}, jpa[3] = {}, x[9] = {};
    double* smp = smp_s[grp];
    long long most = cnt;
    for (int o = 16; o < 64; o <<= 1) most = max(most, (long long)__shfl_xor(most, o, 64));
    for (long long base = 0; base < most; base += 16) {   // uniform
        __syncthreads();   // the samples before have been used
        if (base + c < cnt) {
            const long long s = s0 + base + c;
            double w[3], E[3][3], J[3][3];
            for (int k = 0; k < 3; ++k) w[k] = (gyro[3 * s + k] - b0[k]) * dt;
            so3_exp(w, E);
            right_jacobian(w, J);
            double* o = smp + kPreSample * c;
            for (int r = 0; r < 3; ++r) {
                for (int k = 0; k < 3; ++k) {
                    o[3 * r + k] = E[r][k];
                    o[9 + 3 * r + k] = J[r][k];
                }
                o[18 + r] = acc[3 * s + r] - b0[3 + r];
            }
        }
        __syncthreads();
        const int here = (int)min(16LL, most - base);
        for (int t = 0; t < here; ++t) {   // uniform; a row takes part as a whole
            if (base + t >= cnt) continue;
            const double* o = smp + kPreSample * t;
            double D[3][3], J[3][3], Dc[3], Jc[3], Jr[3], Rr[3];
            for (int r = 0; r < 3; ++r) {
                for (int k = 0; k < 3; ++k) {
                    D[r][k] = o[3 * r + k];
                    J[r][k] = o[9 + 3 * r + k];
                }
                Dc[r] = o[3 * r + c3];
                Jc[r] = o[9 + 3 * r + c3];
                Jr[r] = c < 3 ? o[9 + 3 * c3 + r] * dt : 0.0;
            }
            const double a0 = o[18], a1 = o[19], a2 = o[20];
            double Ra[3], Rax[3][3], Rd[3][3], Rp[3][3];
            for (int r = 0; r < 3; ++r) {
                Ra[r] = dR[r][0] * a0 + dR[r][1] * a1 + dR[r][2] * a2;
                Rax[r][0] = dR[r][1] * a2 - dR[r][2] * a1;
                Rax[r][1] = dR[r][2] * a0 - dR[r][0] * a2;
                Rax[r][2] = dR[r][0] * a1 - dR[r][1] * a0;
                Rr[r] = c3 == 0 ? dR[0][r] : c3 == 1 ? dR[1][r] : dR[2][r];
                for (int k = 0; k < 3; ++k) {
                    Rd[r][k] = -Rax[r][k] * dt;
                    Rp[r][k] = -0.5 * Rax[r][k] * dt * dt;
                }
            }
            // row c of A = [D^T; Rd I; Rp dt I], and of the acceleration
            // noise's matrix [0; R dt; 1/2 R dt^2]
            double Ac[3], Bc[3];
            for (int k = 0; k < 3; ++k) {
                const double d = c3 == 0 ? Rd[0][k] : c3 == 1 ? Rd[1][k] : Rd[2][k];
                const double p = c3 == 0 ? Rp[0][k] : c3 == 1 ? Rp[1][k] : Rp[2][k];
                Ac[k] = c < 3 ? Dc[k] : c < 6 ? d : p;
                Bc[k] = c < 3 ? 0.0 : c < 6 ? Rr[k] * dt : 0.5 * Rr[k] * dt * dt;
            }
            // column c of A cov
            double y[9];
            for (int r = 0; r < 3; ++r) {
                y[r] = D[0][r] * x[0] + D[1][r] * x[1] + D[2][r] * x[2];
                y[3 + r] = Rd[r][0] * x[0] + Rd[r][1] * x[1] + Rd[r][2] * x[2] + x[3 + r];
                y[6 + r] = Rp[r][0] * x[0] + Rp[r][1] * x[1] + Rp[r][2] * x[2] + dt * x[3 + r] + x[6 + r];
            }
            // column c of (A cov) A^T and the noise
            const double near = c >= 6 ? dt : 0.0, same = c >= 3 ? 1.0 : 0.0;
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                double u = row_lane<0>(y[r]) * Ac[0] + row_lane<1>(y[r]) * Ac[1] + row_lane<2>(y[r]) * Ac[2];
                u += SegScan::move<0x113, 0xF>(y[r]) * near;   // row_shr:3
                u += y[r] * same;
                double ng = 0.0, na = 0.0;
                for (int k = 0; k < 3; ++k) {
                    if (r < 3) ng += J[r][k] * dt * Jr[k];
                    else na += (r < 6 ? dR[r - 3][k] * dt : 0.5 * dR[r - 6][k] * dt * dt) * Bc[k];
                }
                x[r] = u + qg * ng + qa * na;
            }
            // bias Jacobians: position, velocity, then rotation
            double rj[3], jr2[3];
            for (int r = 0; r < 3; ++r) {
                rj[r] = Rax[r][0] * jrg[0] + Rax[r][1] * jrg[1] + Rax[r][2] * jrg[2];
                jr2[r] = D[0][r] * jrg[0] + D[1][r] * jrg[1] + D[2][r] * jrg[2];
            }
            for (int r = 0; r < 3; ++r) {
                jpa[r] = jpa[r] + jva[r] * dt - 0.5 * Rc[r] * dt * dt;
                jpg[r] = jpg[r] + jvg[r] * dt - 0.5 * rj[r] * dt * dt;
                jva[r] = jva[r] - Rc[r] * dt;
                jvg[r] = jvg[r] - rj[r] * dt;
                jrg[r] = jr2[r] - Jc[r] * dt;
                dp[r] = dp[r] + dv[r] * dt + 0.5 * Ra[r] * dt * dt;
                dv[r] = dv[r] + Ra[r] * dt;
            }
            for (int r = 0; r < 3; ++r) Rc[r] = dR[r][0] * Dc[0] + dR[r][1] * Dc[1] + dR[r][2] * Dc[2];
            for (int r = 0; r < 3; ++r) {
                dR[r][0] = row_lane<0>(Rc[r]);
                dR[r][1] = row_lane<1>(Rc[r]);
                dR[r][2] = row_lane<2>(Rc[r]);
            }
        }
    }
    if (c < 9)
        for (int r = 0; r < 9; ++r) cov_s[grp][9 * r + c] = x[r];
    __syncthreads();
    if (f >= n) return;
    double* o = out + (size_t)kPreStride * f;
    if (c == 0) {
        o[kDt] = dt * (double)cnt;
        for (int r = 0; r < 3; ++r) {
            o[kDV + r] = dv[r];
            o[kDP + r] = dp[r];
            o[kBg0 + r] = b0[r];
            o[kBa0 + r] = b0[3 + r];
        }
    }
    if (c < 3)
        for (int r = 0; r < 3; ++r) {
            o[kDR + 3 * r + c] = Rc[r];
            o[kJRg + 3 * r + c] = jrg[r];
            o[kJvg + 3 * r + c] = jvg[r];
            o[kJva + 3 * r + c] = jva[r];
            o[kJpg + 3 * r + c] = jpg[r];
            o[kJpa + 3 * r + c] = jpa[r];
        }
    if (c < 9)
        for (int r = 0; r < 9; ++r) o[kCov + 9 * r + c] = 0.5 * (x[r] + cov_s[grp][9 * c + r]);
}

// ------------------------------------------------------------ residuals
// r = (Log((dR Exp(JRg dbg))^T Ri^T Rj),
//      Ri^T (vj - vi - g dt) - (dv + Jvg dbg + Jva dba),
//      Ri^T (pj - pi - vi dt - 1/2 g dt^2) - (dp + Jpg dbg + Jpa dba))
template <typename S>
__device__ __forceinline__ void inertial_residual(const S (&Ri)[3][3], const S (&pi)[3],
                                                  const S (&vi)[3], const S (&bgi)[3],
                                                  const S (&bai)[3], const S (&Rj)[3][3],
                                                  const S (&pj)[3], const S (&vj)[3],
                                                  const double* __restrict__ pre, S (&r)[9]) {
    const double dt = pre[kDt];
    S dbg[3], dba[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        dbg[k] = bgi[k] - pre[kBg0 + k];
        dba[k] = bai[k] - pre[kBa0 + k];
    }
    S corr[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        corr[k] = pre[kJRg + 3 * k] * dbg[0] + pre[kJRg + 3 * k + 1] * dbg[1] + pre[kJRg + 3 * k + 2] * dbg[2];
    S Ec[3][3], dRc[3][3], RiRj[3][3], E[3][3];
    so3_exp(corr, Ec);
    double dR[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) dR[a][b] = pre[kDR + 3 * a + b];
    mm(dR, Ec, dRc);
    mtm(Ri, Rj, RiRj);
    mtm(dRc, RiRj, E);
    S rR[3];
    so3_log(E, rR);
    S wv[3], wp[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        wv[k] = vj[k] - vi[k] - kGravity[k] * dt;
        wp[k] = pj[k] - pi[k] - vi[k] * dt - 0.5 * kGravity[k] * dt * dt;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r[k] = rR[k];
        const S dvc = pre[kDV + k] + (pre[kJvg + 3 * k] * dbg[0] + pre[kJvg + 3 * k + 1] * dbg[1] +
                                      pre[kJvg + 3 * k + 2] * dbg[2]) +
                      (pre[kJva + 3 * k] * dba[0] + pre[kJva + 3 * k + 1] * dba[1] + pre[kJva + 3 * k + 2] * dba[2]);
        const S dpc = pre[kDP + k] + (pre[kJpg + 3 * k] * dbg[0] + pre[kJpg + 3 * k + 1] * dbg[1] +
                                      pre[kJpg + 3 * k + 2] * dbg[2]) +
                      (pre[kJpa + 3 * k] * dba[0] + pre[kJpa + 3 * k + 1] * dba[1] + pre[kJpa + 3 * k + 2] * dba[2]);
        r[3 + k] = Ri[0][k] * wv[0] + Ri[1][k] * wv[1] + Ri[2][k] * wv[2] - dvc;
        r[6 + k] = Ri[0][k] * wp[0] + Ri[1][k] * wp[1] + Ri[2][k] * wp[2] - dpc;
    }
}

// R (I + [d]x): the right perturbation R Exp(d) to first order at d = 0
template <typename S>
__device__ __forceinline__ void perturb_rot(const double (&R)[3][3], const S (&d)[3], S (&Rp)[3][3]) {
    S K[3][3];
    skew(d, K);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            Rp[r][c] = R[r][0] * K[0][c] + R[r][1] * K[1][c] + R[r][2] * K[2][c] + R[r][c];
}

__device__ __forceinline__ void state_rotation(const double* __restrict__ s, double (&R)[3][3]) {
    const double w[3] = {s[0], s[1], s[2]};
    so3_exp(w, R);
}

// One lane per (factor, column): factor f joins keyframes f and f + 1;
// columns dtheta_i, dp_i, dv_i, dbg_i, dba_i, dtheta_j, dp_j, dv_j (3 each).
__global__ __launch_bounds__(256) void k_inertial_eval(int n, const double* __restrict__ st,
                                                       const double* __restrict__ pre,
                                                       double* __restrict__ r_out,
                                                       double* __restrict__ j_out) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= 24LL * n) return;
    const int f = (int)(t / 24), col = (int)(t % 24);
    using S = Dual<double>;
    const double* si = st + 15 * (size_t)f;
    const double* sj = st + 15 * (size_t)(f + 1);
    double Ri0[3][3], Rj0[3][3];
    state_rotation(si, Ri0);
    state_rotation(sj, Rj0);
    S z[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) z[k] = {0.0, k == col ? 1.0 : 0.0};
    S di[3] = {z[0], z[1], z[2]}, dj[3] = {z[15], z[16], z[17]};
    S Ri[3][3], Rj[3][3];
    perturb_rot(Ri0, di, Ri);
    perturb_rot(Rj0, dj, Rj);
    S pi[3], vi[3], bg[3], ba[3], pj[3], vj[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pi[k] = si[3 + k] + z[3 + k];
        vi[k] = si[6 + k] + z[6 + k];
        bg[k] = si[9 + k] + z[9 + k];
        ba[k] = si[12 + k] + z[12 + k];
        pj[k] = sj[3 + k] + z[18 + k];
        vj[k] = sj[6 + k] + z[21 + k];
    }
    S r[9];
    inertial_residual(Ri, pi, vi, bg, ba, Rj, pj, vj, pre + (size_t)kPreStride * f, r);
#pragma unroll
    for (int k = 0; k < 9; ++k) j_out[(size_t)216 * f + 24 * k + col] = r[k].d;
    if (col == 0)
#pragma unroll
        for (int k = 0; k < 9; ++k) r_out[9 * (size_t)f + k] = r[k].v;
}

// One lane per (observation, column): columns dtheta, dp of the keyframe and
// dX of the point.  Xc = R^T (X - p); u_l = fx Xc_x / Xc_z + cx,
// v_l = fy Xc_y / Xc_z + cy, u_r = u_l - fx b / Xc_z; minus the observation.
__global__ __launch_bounds__(256) void k_stereo_eval(long long n, const double* __restrict__ st,
                                                     const double* __restrict__ pts,
                                                     const long long* __restrict__ kf,
                                                     const long long* __restrict__ pt,
                                                     const double* __restrict__ obs, double fx,
                                                     double fy, double cx, double cy, double base,
                                                     double* __restrict__ r_out,
                                                     double* __restrict__ j_out) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= 9LL * n) return;
    const long long e = t / 9;
    const int col = (int)(t % 9);
    using S = Dual<double>;
    const double* s = st + 15 * (size_t)kf[e];
    const double* X = pts + 3 * (size_t)pt[e];
    double R0[3][3];
    state_rotation(s, R0);
    S d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = {0.0, k == col ? 1.0 : 0.0};
    S R[3][3];
    perturb_rot(R0, d, R);
    S q[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const S pk = S{s[3 + k], 3 + k == col ? 1.0 : 0.0};
        const S xk = S{X[k], 6 + k == col ? 1.0 : 0.0};
        q[k] = xk - pk;
    }
    S Xc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) Xc[k] = R[0][k] * q[0] + R[1][k] * q[1] + R[2][k] * q[2];
    const S inv = 1.0 / Xc[2];
    const S ul = fx * Xc[0] * inv + cx;
    const S vl = fy * Xc[1] * inv + cy;
    const S ur = ul - fx * base * inv;
    const S r[3] = {ul - obs[3 * e], vl - obs[3 * e + 1], ur - obs[3 * e + 2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) j_out[(size_t)27 * e + 9 * k + col] = r[k].d;
    if (col == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) r_out[3 * (size_t)e + k] = r[k].v;
}

// block-wide sum of a double over a 256-thread workgroup (lane 0 of the
// first wavefront holds the result)
__device__ __forceinline__ double block_sum_vi(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += red[k];
    return s;
}

// ==========================================================================
// The visual-inertial LM solve (Background Eq. 8; Sec. V-C), FP64
// arithmetic, in two forms of the damped step: the points eliminated (Eq.
// 5-6 on the keyframe / point partition) and PCG on the keyframe Schur
// complement, or the paper's form for its VI runs, PCG on the whole damped
// system over keyframe states and points; block-Jacobi preconditioned
// (15 x 15 keyframe blocks; 3 x 3 point blocks in the whole-system form).
// Unknowns per keyframe: dtheta, dp, dv, dbg, dba (the rotation updated on
// the right); per point: dX.  The first keyframe is held fixed (its columns
// are zero).  Terms:
//   stereo   1/2 rho(|r|^2 / sigma^2), Huber on the squared norm, IRLS
//            whitening sqrt(w) / sigma;
//   inertial 1/2 r^T Omega r, Omega the inverse preintegrated covariance;
//   bias     1/2 r^T Omega_b r, r = b_j - b_i, Omega_b from the random-walk
//            densities and the interval length.
// ==========================================================================
constexpr int kSt = 21;   // device keyframe state: R (row-major), p, v, bg, ba

struct VIDev {
    int K;                 // keyframes
    long long N, M;        // points, stereo observations
    double* st;            // [K kSt] current
    double* st_c;          // [K kSt] candidate
    double* X;             // [3 N]
    double* X_c;
    const int* kf;         // [M]
    const int* pt;
    const double* obs;     // [3 M]
    const double* pre;     // [kPreStride (K - 1)]
    double* info;          // [81 (K - 1)] Omega of the inertial terms
    double* jsp;           // whole-system form: what the stereo Jacobians are made of, the
                           // point in the camera and the whitening factor, in point-order
                           // tiles (js_tile); null in the Schur form
    double* ji;            // [216 (K - 1)] inertial Jacobians
    double* ri;            // [9 (K - 1)]
    double* b;             // [n] gradient J^T Omega r
    double* hk;            // [225 K] keyframe diagonal blocks
    double* hp;            // [9 N] point diagonal blocks
    double* dg;            // [n] clipped diagonal (damping)
    double* mki;           // [225 K] inverses of the damped keyframe blocks (of S in the Schur form)
    double* mp;            // [9 N] inverses of the damped point blocks
    double* scal;          // [8 + kPcgScalars] reductions
    // Schur form (null in the whole-system form): W_e = J_k^T J_p (6 x 3)
    // per observation, in keyframe order (wk) and in padded point order
    // (wp), each in tiles of 64 observations x 18 entries in 16-byte lane
    // groups (w_at)
    void* wk;              // double, or float when w32
    void* wp;
    int w32;
    const int* qkf;        // [Mp] keyframe of the i-th observation in padded point order
    const int* qpt;        // [Mp] its point, -1 in a pad slot
    const double* qobs;    // [3 Mp] the observed pixels in point order
    long long Mp;          // padded point-order length (a multiple of 64)
    const int* longp;      // [nlong] the points with more than 64 observations
    int nlong;
    double* tb;            // [3 N] their partial sums (zero between passes)
    const int* lslot;      // [nlslot] the point-order slots of their observations
    long long nlslot;
    double* sm;            // [36 K] sum over a keyframe's observations of W C^-1 W^T
    // explicit off-diagonal blocks of the Schur complement's visual part
    // (null when the products stay implicit): the covisible keyframes of each
    // keyframe in ascending order, their 6 x 6 blocks -sum W C^-1 W^T, and for
    // the blocks of a later keyframe the pairs of point-order slots they sum
    const int* kslot;      // [M] point-order slot of each keyframe-order observation
    const int* kinv;       // [Mp] and back
    const int* kfoff;      // [K + 1] keyframe-order range of each keyframe
    int* nrow;             // [K + 2] (the last: observations far from their workgroup's keyframes)
    int* nitem;            // [K + 1] first pair of each keyframe
    int* ncol;             // [nnz]
    int* noff;             // [nnz] first pair of each block (later keyframes; the others unused)
    int* nkf;              // [nnz] the block's own keyframe
    int nnz;
    int2* items;           // pairs of keyframe-order observations
    double* vblk;          // [36 nnz]
    double* ad;            // [225 K] damped diagonal blocks of S
    double* cb;            // [225 (K - 1)] cross blocks of consecutive keyframes (inertial and
    double* cbt;           // bias terms), and transposed
    double* icx;           // [135 (K - 1)] inertial cross blocks J_i^T Omega J_j (15 x 9)
    double fx, fy, cx, cy, base, inv_sigma, delta2, wg, wa;   // wg, wa: 1 / sigma_w^2
};

// PCG scalars on the device: three slots of dot accumulators {p.q parts,
// r.r, r.z, ...}, used round robin (step s accumulates into slot s % 3,
// takes the previous step's values from slot (s + 2) % 3 and clears slot
// (s + 1) % 3 for the next step, so no kernel reads a value another
// workgroup of it resets), then the stop threshold, the stop flag, the step
// count and the squared rejection ratio
// p.q is summed in kPqParts parts (a workgroup adds to part blockIdx %
// kPqParts: thousands of workgroups adding to one address serialise)
constexpr int kPqParts = 256;
// per slot also: the least r.r so far (the rejection test), a breakdown flag
// set by the update kernel and the stop decision of the direction kernel
enum { kAccPq = 0, kAccRr = kPqParts, kAccRz, kAccMin, kAccBreak, kAccStop, kAccRrP,
       kAccRzP = kAccRrP + kPqParts, kAccN = kAccRzP + kPqParts };
constexpr int kSlots = 3;
enum { kThr = kSlots * kAccN, kDone, kSteps, kRatio2, kPcgScalars };
// the cost, |x| and model-decrease sums: kRedSlots sums of kPqParts parts
// each, after the PCG scalars (scal = 8 unused, the PCG scalars, the parts)
// (the step kernel's sums, then the cross term and the cost)
constexpr int kRedSlots = 8, kStepSums = 5;
enum { kRedQuad = 0, kRedBp, kRedB, kRedDx, kRedX, kRedCross, kRedCost };
constexpr long long kRedOff = 8 + kPcgScalars;
constexpr long long kScalN = kRedOff + (long long)kRedSlots * kPqParts;

__device__ __forceinline__ bool pcg_done(const double* ps) { return ps && ps[kDone] != 0.0; }

// the keyframe window of the LDS partials of the point-order products, and
// their workgroup size
constexpr int kKfWin = 64;
constexpr int kFuseBlock = 512;

// W tiles: 64 observations x 18 entries, in 16-byte groups so that a lane
// loads its entries as float4 / double2 and one load instruction of a
// wavefront reads 1 KiB contiguous: group g (V = 16 / sizeof(WT) entries,
// the last one of FP32 two wide) of lane l at tile + 64 V g + width l
template <typename WT>
__device__ __forceinline__ size_t w_at(long long e, int c) {
    constexpr int V = 16 / (int)sizeof(WT);
    const int g = c / V;
    const int width = (18 - g * V) < V ? (18 - g * V) : V;
    return (size_t)(e >> 6) * (18 * 64) + (size_t)g * V * 64 + (size_t)(e & 63) * width + (c - g * V);
}

template <typename WT>
__device__ __forceinline__ void load_w(const void* w, long long e, double (&out)[18]);

template <>
__device__ __forceinline__ void load_w<float>(const void* w, long long e, double (&out)[18]) {
    const float* t = (const float*)w + (size_t)(e >> 6) * (18 * 64);
    const int l = (int)(e & 63);
    for (int g = 0; g < 4; ++g) {
        const float4 v = ((const float4*)t)[g * 64 + l];
        out[4 * g] = v.x;
        out[4 * g + 1] = v.y;
        out[4 * g + 2] = v.z;
        out[4 * g + 3] = v.w;
    }
    const float2 v = ((const float2*)(t + 1024))[l];
    out[16] = v.x;
    out[17] = v.y;
}

template <>
__device__ __forceinline__ void load_w<double>(const void* w, long long e, double (&out)[18]) {
    const double* t = (const double*)w + (size_t)(e >> 6) * (18 * 64);
    const int l = (int)(e & 63);
    for (int g = 0; g < 9; ++g) {
        const double2 v = ((const double2*)t)[g * 64 + l];
        out[2 * g] = v.x;
        out[2 * g + 1] = v.y;
    }
}

__device__ __forceinline__ void atomic_add(double* a, double v) { unsafeAtomicAdd(a, v); }

__global__ void k_vi_states_in(int K, const double* __restrict__ s15, double* __restrict__ s21) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const double w[3] = {s15[15 * k], s15[15 * k + 1], s15[15 * k + 2]};
    double R[3][3];
    so3_exp(w, R);
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) s21[kSt * k + 3 * r + c] = R[r][c];
    for (int j = 0; j < 12; ++j) s21[kSt * k + 9 + j] = s15[15 * k + 3 + j];
}

__global__ void k_vi_states_out(int K, const double* __restrict__ s21, double* __restrict__ s15) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    double R[3][3], w[3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) R[r][c] = s21[kSt * k + 3 * r + c];
    so3_log(R, w);
    for (int j = 0; j < 3; ++j) s15[15 * k + j] = w[j];
    for (int j = 0; j < 12; ++j) s15[15 * k + 3 + j] = s21[kSt * k + 9 + j];
}

// Omega = cov^-1 per interval by Cholesky (cov = L L^T): Omega = L^-T L^-1.
__global__ void k_vi_info(int n, const double* __restrict__ pre, double* __restrict__ info) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= n) return;
    const double* C = pre + (size_t)kPreStride * f + kCov;
    double L[9][9] = {};
    for (int j = 0; j < 9; ++j) {
        double d = C[9 * j + j];
        for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
        L[j][j] = sqrt(d);
        for (int i = j + 1; i < 9; ++i) {
            double t = C[9 * i + j];
            for (int k = 0; k < j; ++k) t -= L[i][k] * L[j][k];
            L[i][j] = t / L[j][j];
        }
    }
    double Li[9][9] = {};   // L^-1 (lower)
    for (int c = 0; c < 9; ++c) {
        for (int r = c; r < 9; ++r) {
            double t = r == c ? 1.0 : 0.0;
            for (int k = c; k < r; ++k) t -= L[r][k] * Li[k][c];
            Li[r][c] = t / L[r][r];
        }
    }
    double* O = info + 81 * (size_t)f;
    for (int r = 0; r < 9; ++r)
        for (int c = 0; c < 9; ++c) {
            double t = 0.0;
            for (int k = (r > c ? r : c); k < 9; ++k) t += Li[k][r] * Li[k][c];
            O[9 * r + c] = t;
        }
}

// Stereo projection of observation e at (R, p) and X: Xc, the prediction and
// (with kJac) the 3 x 9 Jacobian over dtheta, dp, dX.
template <bool kJac>
__device__ __forceinline__ void vi_stereo(const VIDev& d, const double* __restrict__ s,
                                          const double* __restrict__ X, long long e, double (&r)[3],
                                          double (&J)[3][9], double (&Xc)[3]) {
    double q[3];
    for (int k = 0; k < 3; ++k) q[k] = X[k] - s[9 + k];
    for (int k = 0; k < 3; ++k) Xc[k] = s[k] * q[0] + s[3 + k] * q[1] + s[6 + k] * q[2];
    const double iz = 1.0 / Xc[2];
    const double ul = d.fx * Xc[0] * iz + d.cx;
    r[0] = ul - d.obs[3 * e];
    r[1] = d.fy * Xc[1] * iz + d.cy - d.obs[3 * e + 1];
    r[2] = ul - d.fx * d.base * iz - d.obs[3 * e + 2];
    if (!kJac) return;
    double P[3][3] = {{d.fx * iz, 0.0, -d.fx * Xc[0] * iz * iz},
                      {0.0, d.fy * iz, -d.fy * Xc[1] * iz * iz},
                      {d.fx * iz, 0.0, -d.fx * (Xc[0] - d.base) * iz * iz}};
    const double Kx[3][3] = {{0.0, -Xc[2], Xc[1]}, {Xc[2], 0.0, -Xc[0]}, {-Xc[1], Xc[0], 0.0}};
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) {
            J[a][c] = P[a][0] * Kx[0][c] + P[a][1] * Kx[1][c] + P[a][2] * Kx[2][c];
            // P R^T: (R^T)[k][c] = R[c][k]
            const double PRt = P[a][0] * s[3 * c] + P[a][1] * s[3 * c + 1] + P[a][2] * s[3 * c + 2];
            J[a][3 + c] = -PRt;
            J[a][6 + c] = PRt;
        }
}

__device__ __forceinline__ void vi_huber(double s, double delta2, double& rho, double& w) {
    if (delta2 > 0.0 && s > delta2) {
        const double q = sqrt(s);
        rho = 2.0 * sqrt(delta2) * q - delta2;
        w = sqrt(delta2) / q;
    } else {
        rho = s;
        w = 1.0;
    }
}

// whitened residual and Jacobian of observation (k, j) with the observed
// pixels ob (zero when !valid; the first keyframe's columns zero); jc: the
// point in the camera and the whitening factor
__device__ __forceinline__ void vi_stereo_whitened(const VIDev& d, const double* __restrict__ ob, int k, int j,
                                                   bool valid, double (&r)[3], double (&J)[3][9],
                                                   double (&jc)[4]) {
    VIDev dd = d;
    dd.obs = ob;
    double Xc[3];
    vi_stereo<true>(dd, d.st + (size_t)kSt * k, d.X + 3 * (size_t)j, 0, r, J, Xc);
    const double s = (r[0] * r[0] + r[1] * r[1] + r[2] * r[2]) * d.inv_sigma * d.inv_sigma;
    double rho, w;
    vi_huber(s, d.delta2, rho, w);
    const double sc = valid ? sqrt(w) * d.inv_sigma : 0.0;
    for (int a = 0; a < 3; ++a) jc[a] = Xc[a];
    jc[3] = sc;
    for (int a = 0; a < 3; ++a) {
        r[a] *= sc;
        for (int c = 0; c < 9; ++c) J[a][c] = (k == 0 && c < 6) ? 0.0 : J[a][c] * sc;
    }
}

// linearisation of the stereo terms in keyframe order: the keyframe's
// gradient and 6 x 6 block terms summed across its run of the wavefront
// (SegScan) and added once per run; in the Schur form W = J_k^T J_p is
// stored (keyframe-order tiles).  The point terms come from the point-order
// pass below.
__global__ void k_vi_lin_stereo(VIDev d) {
    const long long e0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const bool valid = e0 < d.M;
    const long long e = valid ? e0 : d.M - 1;
    const int k = d.kf[e], j = d.pt[e];
    const int l = (int)(threadIdx.x & 63);
    const int kprev = __shfl_up(k, 1, 64);
    const bool start = !valid || l == 0 || kprev != k;
    const SegScan seg(start);
    int head, end;
    segment_of(__ballot(start), l, head, end);
    double r[3], J[3][9], jc[4];
    vi_stereo_whitened(d, d.obs + 3 * e, k, j, valid, r, J, jc);
    if (valid && d.wk)
        for (int a = 0; a < 6; ++a)
            for (int c = 0; c < 3; ++c) {
                const double w = J[0][a] * J[0][6 + c] + J[1][a] * J[1][6 + c] + J[2][a] * J[2][6 + c];
                if (d.w32) ((float*)d.wk)[w_at<float>(e, 3 * a + c)] = (float)w;
                else ((double*)d.wk)[w_at<double>(e, 3 * a + c)] = w;
            }
    const bool last = valid && l == end;
    double* bk = d.b + 15 * (size_t)k;
    for (int c = 0; c < 6; ++c) {
        const double sg = seg.sum(J[0][c] * r[0] + J[1][c] * r[1] + J[2][c] * r[2]);
        if (last) atomic_add(bk + c, sg);
    }
    for (int a = 0; a < 6; ++a)
        for (int c = a; c < 6; ++c) {
            const double h = seg.sum(J[0][a] * J[0][c] + J[1][a] * J[1][c] + J[2][a] * J[2][c]);
            if (last && k != 0) {
                atomic_add(d.hk + 225 * (size_t)k + 15 * a + c, h);
                if (c != a) atomic_add(d.hk + 225 * (size_t)k + 15 * c + a, h);
            }
        }
}

// the whole-system form's stereo terms in padded point-order tiles of 64
// slots: the point in the camera (3 x 64 doubles), then the whitening factors
// (64 doubles, or floats when w32: a row of the Jacobian then carries one FP32
// rounding, as each of its entries did when it was stored)
__device__ __forceinline__ double* js_tile(const VIDev& d, long long i) {
    return d.jsp + (size_t)(i >> 6) * (d.w32 ? 224 : 256);
}
__device__ __forceinline__ void js_save(const VIDev& d, long long i, const double (&jc)[4]) {
    double* t = js_tile(d, i);
    const int l = (int)(i & 63);
    for (int c = 0; c < 3; ++c) t[64 * c + l] = jc[c];
    if (d.w32) ((float*)(t + 192))[l] = (float)jc[3];
    else t[192 + l] = jc[3];
}
__device__ __forceinline__ void js_load(const VIDev& d, long long i, double (&jc)[4]) {
    const double* t = js_tile(d, i);
    const int l = (int)(i & 63);
    for (int c = 0; c < 3; ++c) jc[c] = t[64 * c + l];
    jc[3] = d.w32 ? (double)((const float*)(t + 192))[l] : t[192 + l];
}

// the same terms in point order: W (Schur form) or the Jacobian's terms
// (whole-system form) stored in point-order tiles,
// the point's gradient b_p and block H_pp summed across its run of the
// wavefront; a point whose observations all sit in one wavefront is stored,
// one split across wavefronts is added in parts (b and hp are zero before)
template <typename WT>
__global__ void k_vi_lin_stereo_pts(VIDev d) {
    const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long i = i0 < d.Mp ? i0 : d.Mp - 1;
    const int jq = d.qpt[i];
    const bool valid = i0 < d.Mp && jq >= 0;
    const int j = valid ? jq : 0, k = valid ? d.qkf[i] : 0;
    const int l = (int)(threadIdx.x & 63);
    const int jprev = __shfl_up(jq, 1, 64);
    const bool start = !valid || l == 0 || jprev != jq;
    const SegScan seg(start);
    int head, end;
    segment_of(__ballot(start), l, head, end);
    const bool first = i == 0 || d.qpt[i - 1] != jq;
    const bool lastp = i == d.Mp - 1 || d.qpt[i + 1] != jq;
    const bool whole = (__shfl(first ? 1 : 0, head, 64) != 0) && lastp;
    double r[3], J[3][9], jc[4];
    vi_stereo_whitened(d, d.qobs + 3 * i, k, j, valid, r, J, jc);
    if (valid && d.wp)
        for (int a = 0; a < 6; ++a)
            for (int c = 0; c < 3; ++c)
                ((WT*)d.wp)[w_at<WT>(i, 3 * a + c)] =
                    (WT)(J[0][a] * J[0][6 + c] + J[1][a] * J[1][6 + c] + J[2][a] * J[2][6 + c]);
    if (d.jsp && i0 < d.Mp) {
        const double pad[4] = {0.0, 0.0, 1.0, 0.0};
        double js[4];
        for (int c = 0; c < 4; ++c) js[c] = valid ? jc[c] : pad[c];
        js_save(d, i, js);
    }
    const bool out = valid && l == end;
    double* bp = d.b + 15 * (size_t)d.K + 3 * (size_t)j;
    for (int c = 0; c < 3; ++c) {
        const double g = seg.sum(J[0][6 + c] * r[0] + J[1][6 + c] * r[1] + J[2][6 + c] * r[2]);
        if (out) {
            if (whole) bp[c] = g;
            else atomic_add(bp + c, g);
        }
    }
    double* hp = d.hp + 9 * (size_t)j;
    for (int a = 0; a < 3; ++a)
        for (int c = a; c < 3; ++c) {
            const double h = seg.sum(J[0][6 + a] * J[0][6 + c] + J[1][6 + a] * J[1][6 + c] +
                                     J[2][6 + a] * J[2][6 + c]);
            if (!out) continue;
            if (whole) {
                hp[3 * a + c] = h;
                hp[3 * c + a] = h;
            } else {
                atomic_add(hp + 3 * a + c, h);
                if (c != a) atomic_add(hp + 3 * c + a, h);
            }
        }
}

// inertial Jacobians by forward-mode AD, one lane per (term, column), at the
// device states (rotation matrices); columns of a fixed first keyframe zero
__global__ __launch_bounds__(256) void k_vi_lin_inertial(VIDev d) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const int n = d.K - 1;
    if (t >= 24LL * n) return;
    const int f = (int)(t / 24), col = (int)(t % 24);
    using S = Dual<double>;
    const double* si = d.st + (size_t)kSt * f;
    const double* sj = d.st + (size_t)kSt * (f + 1);
    double Ri0[3][3], Rj0[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            Ri0[r][c] = si[3 * r + c];
            Rj0[r][c] = sj[3 * r + c];
        }
    S z[24];
    for (int k = 0; k < 24; ++k) z[k] = {0.0, k == col ? 1.0 : 0.0};
    S di[3] = {z[0], z[1], z[2]}, dj[3] = {z[15], z[16], z[17]};
    S Ri[3][3], Rj[3][3];
    perturb_rot(Ri0, di, Ri);
    perturb_rot(Rj0, dj, Rj);
    S pi[3], vi_[3], bg[3], ba[3], pj[3], vj[3];
    for (int k = 0; k < 3; ++k) {
        pi[k] = si[9 + k] + z[3 + k];
        vi_[k] = si[12 + k] + z[6 + k];
        bg[k] = si[15 + k] + z[9 + k];
        ba[k] = si[18 + k] + z[12 + k];
        pj[k] = sj[9 + k] + z[18 + k];
        vj[k] = sj[12 + k] + z[21 + k];
    }
    S r[9];
    inertial_residual(Ri, pi, vi_, bg, ba, Rj, pj, vj, d.pre + (size_t)kPreStride * f, r);
    const bool zero = f == 0 && col < 15;
    for (int k = 0; k < 9; ++k) d.ji[(size_t)216 * f + 24 * k + col] = zero ? 0.0 : r[k].d;
    if (col == 0)
        for (int k = 0; k < 9; ++k) d.ri[9 * (size_t)f + k] = r[k].v;
}

// inertial and bias terms: gradient and diagonal blocks, one wavefront per
// term, lane c < 24 for column c (keyframe i's 15, then keyframe j's first 9)
__global__ __launch_bounds__(256) void k_vi_acc_inertial(VIDev d) {
    const int f = (int)((blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6);
    const int l = (int)(threadIdx.x & 63);
    if (f >= d.K - 1) return;   // whole wavefronts
    const double* J = d.ji + (size_t)216 * f;
    const double* O = d.info + 81 * (size_t)f;
    const double* r = d.ri + 9 * (size_t)f;
    double* bi = d.b + 15 * (size_t)f;
    double* bj = d.b + 15 * (size_t)(f + 1);
    double* hi = d.hk + 225 * (size_t)f;
    double* hj = d.hk + 225 * (size_t)(f + 1);
    if (l < 24) {
        double Or[9], OJ[9];   // Omega r, and column l of Omega J
        for (int a = 0; a < 9; ++a) {
            double t = 0.0, u = 0.0;
            for (int c = 0; c < 9; ++c) {
                t += O[9 * a + c] * r[c];
                u += O[9 * a + c] * J[24 * c + l];
            }
            Or[a] = t;
            OJ[a] = u;
        }
        double g = 0.0;
        for (int a = 0; a < 9; ++a) g += J[24 * a + l] * Or[a];
        atomic_add(l < 15 ? bi + l : bj + (l - 15), g);
        // column l of J^T Omega J within its keyframe's block
        const int c0 = l < 15 ? 0 : 15, c1 = l < 15 ? 15 : 24;
        for (int c = c0; c < c1; ++c) {
            double t = 0.0;
            for (int a = 0; a < 9; ++a) t += J[24 * a + c] * OJ[a];
            if (l < 15) atomic_add(hi + 15 * c + l, t);
            else atomic_add(hj + 15 * (c - 15) + (l - 15), t);
        }
    } else if (l < 30) {
        // bias random walk: r = b_j - b_i (6), Omega_b = diag(wg I3, wa I3) / dt
        const int k = l - 24;
        const double dt = d.pre[(size_t)kPreStride * f + kDt];
        const double* si = d.st + (size_t)kSt * f;
        const double* sj = d.st + (size_t)kSt * (f + 1);
        const double w = (k < 3 ? d.wg : d.wa) / dt;
        const double rb = sj[15 + k] - si[15 + k];
        atomic_add(bj + 9 + k, w * rb);
        atomic_add(hj + 15 * (9 + k) + 9 + k, w);
        if (f != 0) {
            atomic_add(bi + 9 + k, -w * rb);
            atomic_add(hi + 15 * (9 + k) + 9 + k, w);
        }
    }
}

// cost at (st, X): 1/2 sum rho over stereo, 1/2 r^T Omega r over inertial,
// 1/2 r^T Omega_b r over bias; into the parts of reduction slot `slot`
__global__ void k_vi_cost(VIDev d, const double* __restrict__ st, const double* __restrict__ X,
                          int slot) {
    __shared__ double red[16];
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    double c = 0.0;
    if (t < d.M) {
        double r[3], J[3][9], Xc[3];
        vi_stereo<false>(d, st + (size_t)kSt * d.kf[t], X + 3 * (size_t)d.pt[t], t, r, J, Xc);
        double rho, w;
        vi_huber((r[0] * r[0] + r[1] * r[1] + r[2] * r[2]) * d.inv_sigma * d.inv_sigma, d.delta2, rho, w);
        c = 0.5 * rho;
    } else if (t < d.M + d.K - 1) {
        const int f = (int)(t - d.M);
        const double* si = st + (size_t)kSt * f;
        const double* sj = st + (size_t)kSt * (f + 1);
        double Ri[3][3], Rj[3][3], pi[3], vi_[3], bg[3], ba[3], pj[3], vj[3];
        for (int a = 0; a < 3; ++a) {
            for (int b = 0; b < 3; ++b) {
                Ri[a][b] = si[3 * a + b];
                Rj[a][b] = sj[3 * a + b];
            }
            pi[a] = si[9 + a];
            vi_[a] = si[12 + a];
            bg[a] = si[15 + a];
            ba[a] = si[18 + a];
            pj[a] = sj[9 + a];
            vj[a] = sj[12 + a];
        }
        double r[9];
        inertial_residual(Ri, pi, vi_, bg, ba, Rj, pj, vj, d.pre + (size_t)kPreStride * f, r);
        const double* O = d.info + 81 * (size_t)f;
        for (int a = 0; a < 9; ++a)
            for (int b = 0; b < 9; ++b) c += 0.5 * r[a] * O[9 * a + b] * r[b];
        const double dt = d.pre[(size_t)kPreStride * f + kDt];
        for (int k = 0; k < 6; ++k) {
            const double rb = sj[15 + k] - si[15 + k];
            c += 0.5 * ((k < 3 ? d.wg : d.wa) / dt) * rb * rb;
        }
    }
    c = block_sum_vi(c, red);
    if (threadIdx.x == 0) atomic_add(d.scal + kRedOff + slot * kPqParts + blockIdx.x % kPqParts, c);
}

// arrays to be cleared in one launch
struct ZeroList {
    static constexpr int kMax = 6;
    double* p[kMax] = {};
    long long n[kMax] = {};
    int used = 0;
    void add(double* q, long long len) {
        p[used] = q;
        n[used++] = len;
    }
    long long total() const {
        long long s = 0;
        for (int i = 0; i < used; ++i) s += n[i];
        return s;
    }
    __device__ __forceinline__ void clear(long long t) const {
#pragma unroll
        for (int i = 0; i < kMax; ++i) {
            if (t >= 0 && t < n[i]) p[i][t] = 0.0;
            t -= n[i];
        }
    }
};

__global__ void k_vi_clear(ZeroList zero) {
    zero.clear(blockIdx.x * (long long)blockDim.x + threadIdx.x);
}

// (A trial's kernels around the PCG take 1-15 us each at a few thousand
// observations, so launches and readbacks count: 22 launches and one readback
// where it had 40 and three; 31 keyframes: the solve from 5.1 to 4.5 ms.)
// the start of a damped step: the point blocks of the preconditioner (and,
// in the Schur form, C^-1): D = clip(diag H_pp), the damped 3 x 3 block
// inverted by cofactors, one lane per point, and with zb -C^-1 b_p; r = -b
// over nr unknowns; and what the step adds into or starts from zero
__global__ void k_vi_begin(VIDev d, double lam, double lo, double hi, long long nr, double* __restrict__ r,
                           double* __restrict__ zb, ZeroList zero) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= d.N + nr) {
        zero.clear(t - d.N - nr);
    } else if (t >= d.N) {
        r[t - d.N] = -d.b[t - d.N];
    } else {
        const long long j = t;
        const double* H = d.hp + 9 * j;
        double A[3][3];
        for (int a = 0; a < 3; ++a) {
            const double dd = fmin(fmax(H[4 * a], lo), hi);
            d.dg[15 * (size_t)d.K + 3 * j + a] = dd;
            for (int c = 0; c < 3; ++c) A[a][c] = H[3 * a + c] + (a == c ? lam * dd : 0.0);
        }
        const double c00 = A[1][1] * A[2][2] - A[1][2] * A[2][1];
        const double c01 = A[1][2] * A[2][0] - A[1][0] * A[2][2];
        const double c02 = A[1][0] * A[2][1] - A[1][1] * A[2][0];
        const double det = A[0][0] * c00 + A[0][1] * c01 + A[0][2] * c02;
        const double id = 1.0 / det;
        double* M = d.mp + 9 * j;
        M[0] = c00 * id;
        M[1] = (A[0][2] * A[2][1] - A[0][1] * A[2][2]) * id;
        M[2] = (A[0][1] * A[1][2] - A[0][2] * A[1][1]) * id;
        M[3] = c01 * id;
        M[4] = (A[0][0] * A[2][2] - A[0][2] * A[2][0]) * id;
        M[5] = (A[0][2] * A[1][0] - A[0][0] * A[1][2]) * id;
        M[6] = c02 * id;
        M[7] = (A[0][1] * A[2][0] - A[0][0] * A[2][1]) * id;
        M[8] = (A[0][0] * A[1][1] - A[0][1] * A[1][0]) * id;
        if (zb) {
            const double* bp = d.b + 15 * (size_t)d.K + 3 * j;
            for (int a = 0; a < 3; ++a)
                zb[3 * j + a] = -(M[3 * a] * bp[0] + M[3 * a + 1] * bp[1] + M[3 * a + 2] * bp[2]);
        }
    }
}

// the keyframe blocks of the preconditioner, one wavefront per keyframe:
// D = clip(diag H), A = H + lambda diag(D) (less sm in the Schur form),
// factored A = L L^T in LDS (right-looking, the trailing update spread over
// the lanes), then A^-1 column by column (lane c < 15 solves L L^T x = e_c)
__global__ __launch_bounds__(256) void k_vi_precond_kf(VIDev d, double lam, double lo, double hi) {
    __shared__ double La[4][225];
    const int w = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
    const long long k = blockIdx.x * 4LL + w;
    if (k >= d.K) return;   // whole wavefronts; no workgroup barrier below
    double* A = La[w];
    const double* H = d.hk + 225 * (size_t)k;
    for (int e = l; e < 225; e += 64) {
        const int a = e / 15, c = e % 15;
        double v = H[e];
        if (a == c) {
            const double dd = fmin(fmax(v, lo), hi);
            d.dg[15 * (size_t)k + a] = dd;
            v += lam * dd;
        }
        if (d.sm && a < 6 && c < 6) v -= d.sm[36 * (size_t)k + 6 * a + c];
        if (d.ad) d.ad[225 * (size_t)k + e] = v;   // the explicit products' diagonal block
        A[e] = v;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int j = 0; j < 15; ++j) {
        const double ljj = sqrt(fmax(A[16 * j], 1e-300));
        if (l > j && l < 15) A[15 * l + j] /= ljj;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (l == 0) A[16 * j] = ljj;
        // trailing update of the lower triangle: (a, c), j < c <= a < 15
        for (int e = l; e < 225; e += 64) {
            const int a = e / 15, c = e % 15;
            if (c > j && c <= a) A[e] -= A[15 * a + j] * A[15 * c + j];
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    if (l < 15) {
        double y[15];
        for (int i = 0; i < 15; ++i) {
            double u = i == l ? 1.0 : 0.0;
            for (int q = 0; q < i; ++q) u -= A[15 * i + q] * y[q];
            y[i] = u / A[16 * i];
        }
        for (int i = 14; i >= 0; --i) {
            double u = y[i];
            for (int q = i + 1; q < 15; ++q) u -= A[15 * q + i] * y[q];
            y[i] = u / A[16 * i];
        }
        double* Mi = d.mki + 225 * (size_t)k;
        for (int i = 0; i < 15; ++i) Mi[15 * i + l] = y[i];
    }
}

// z = M^-1 r: one lane per keyframe row (the block inverse's row times the
// keyframe's residual), one per point of the first npt; the first direction
// p = z, and r.r and r.z into the parts of acc
__global__ __launch_bounds__(256) void k_vi_apply_m(VIDev d, long long npt, const double* __restrict__ r,
                                                   double* __restrict__ z, double* __restrict__ p,
                                                   double* __restrict__ acc) {
    __shared__ double red[16];
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    double rr = 0.0, rz = 0.0;
    if (t < 15LL * d.K) {
        const long long k = t / 15;
        const int row = (int)(t % 15);
        const double* Mi = d.mki + 225 * (size_t)k + 15 * row;
        const double* rk = r + 15 * (size_t)k;
        double u = 0.0;
        for (int c = 0; c < 15; ++c) u += Mi[c] * rk[c];
        z[t] = u;
        p[t] = u;
        rr = rk[row] * rk[row];
        rz = rk[row] * u;
    } else if (t < 15LL * d.K + npt) {
        const long long j = t - 15LL * d.K;
        const size_t o = 15 * (size_t)d.K + 3 * j;
        const double* M = d.mp + 9 * j;
        const double a = r[o], b = r[o + 1], c = r[o + 2];
        for (int i = 0; i < 3; ++i) {
            const double u = M[3 * i] * a + M[3 * i + 1] * b + M[3 * i + 2] * c;
            z[o + i] = u;
            p[o + i] = u;
            rr += r[o + i] * r[o + i];
            rz += r[o + i] * u;
        }
    }
    rr = block_sum_vi(rr, red);
    __syncthreads();
    rz = block_sum_vi(rz, red);
    if (threadIdx.x == 0) {
        atomic_add(acc + kAccRrP + blockIdx.x % kPqParts, rr);
        atomic_add(acc + kAccRzP + blockIdx.x % kPqParts, rz);
    }
}

// ---- Schur form: the points eliminated (Eq. 5-6 on the keyframe / point
// partition).  With the damped blocks A (keyframes), B (keyframe-point,
// B_kj = W_e for the observation e of point j in keyframe k) and C (points):
//   S p = A p - B C^-1 B^T p,  v = -b_k + B C^-1 b_p,
//   x_p = C^-1 (-b_p - B^T x_k).
// A p is the keyframe diagonal blocks (hk + lambda D) plus the inertial and
// bias cross terms between consecutive keyframes.

// row t of A v: the keyframe diagonal block (damped) and the cross blocks to
// keyframes k - 1 and k + 1 (inertial, and the bias random walk's -Omega_b)
__device__ __forceinline__ double vi_ap_row(const VIDev& d, double lam, const double* __restrict__ v, long long t) {
    const long long k = t / 15;
    const int row = (int)(t % 15);
    const double* H = d.hk + 225 * (size_t)k + 15 * row;
    const double* vk = v + 15 * (size_t)k;
    double u = lam * d.dg[t] * vk[row];
    for (int c = 0; c < 15; ++c) u += H[c] * vk[c];
    if (k + 1 < d.K) {   // keyframe k as i of the term k: row of icx_k
        const double* C = d.icx + 135 * (size_t)k + 9 * row;
        const double* vj = v + 15 * (size_t)(k + 1);
        for (int c = 0; c < 9; ++c) u += C[c] * vj[c];
        if (row >= 9 && k != 0) {
            const double dt = d.pre[(size_t)kPreStride * k + kDt];
            u -= ((row < 12 ? d.wg : d.wa) / dt) * vj[row];
        }
    }
    if (k > 0) {         // keyframe k as j of the term k - 1: column of icx_{k-1}
        const double* vi = v + 15 * (size_t)(k - 1);
        if (row < 9) {
            const double* C = d.icx + 135 * (size_t)(k - 1) + row;
            for (int c = 0; c < 15; ++c) u += C[9 * c] * vi[c];
        } else if (k - 1 != 0) {
            const double dt = d.pre[(size_t)kPreStride * (k - 1) + kDt];
            u -= ((row < 12 ? d.wg : d.wa) / dt) * vi[row];
        }
    }
    return u;
}

// z_j = sign C_j^-1 (sum_{e of j} W_e^T v_k(e) + add_j): observations in
// padded point order (a point's observations within one wavefront unless it
// has more than 64; pad slots have point -1), a point's sum across its run of
// the wavefront.  A whole run stores z_j and, with acc, adds -t_j . z_j to
// acc (the point part of p . S p = p . A p - sum_j t_j . C_j^-1 t_j); a run
// of a point split across wavefronts adds its part of t_j to tb for
// k_vi_long_pts
//
// kFuse (the PCG product, sign 1, no add): the keyframe side too, q_k -=
// sum_{e of k} W_e z_j(e), in the same pass: z_j goes from the run's last
// lane to the run, each observation's W_e z_j is added to the workgroup's
// LDS partials of the keyframes kbase .. kbase + kKfWin - 1 (kbase the least
// keyframe the workgroup sees; points are numbered by first observing
// keyframe, so a workgroup's keyframes lie close together; one further out
// is added to q directly), and the partials go to q with one atomic add
// each.  Split points take this step in k_vi_long_kf.  The workgroups after
// the point ones add q += A v (one lane per keyframe row, vi_ap_row; q is
// zero beforehand) and v . A v: the whole product S v in one launch.

template <typename WT, bool kFuse>
__global__ __launch_bounds__(1024) void k_vi_schur_pts(VIDev d, const double* __restrict__ v,
                                                      const double* __restrict__ add, double sign,
                                                      double* __restrict__ z, const double* __restrict__ ps,
                                                      double* __restrict__ acc, double* __restrict__ q,
                                                      double lam) {
    if (pcg_done(ps)) return;
    __shared__ double red[16];
    __shared__ double part[kFuse ? kKfWin * 6 : 1];
    __shared__ int kmin_w[16];
    if (kFuse) {
        const long long pt_blocks = (d.Mp + blockDim.x - 1) / blockDim.x;
        if (blockIdx.x >= pt_blocks) {   // the keyframe rows (uniform per workgroup)
            const long long t0 = (blockIdx.x - pt_blocks) * (long long)blockDim.x + threadIdx.x;
            const bool act = t0 < 15LL * d.K;
            const long long t = act ? t0 : 0;
            const double u = vi_ap_row(d, lam, v, t);
            if (act) atomic_add(q + t, u);
            const double sa = block_sum_vi(act ? v[t] * u : 0.0, red);
            if (threadIdx.x == 0) atomic_add(acc + blockIdx.x % kPqParts, sa);
            return;
        }
    }
    const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long i = i0 < d.Mp ? i0 : d.Mp - 1;
    const int j = d.qpt[i];
    const bool valid = i0 < d.Mp && j >= 0;
    const int jj = valid ? j : 0, k = valid ? d.qkf[i] : 0;
    const int l = (int)(threadIdx.x & 63);
    const int jprev = __shfl_up(j, 1, 64);
    const bool start = !valid || l == 0 || jprev != j;
    const SegScan seg(start);
    int head, end;
    segment_of(__ballot(start), l, head, end);
    // the point's first and last observations in the whole order
    const bool first = i == 0 || d.qpt[i - 1] != j;
    const bool last = i == d.Mp - 1 || d.qpt[i + 1] != j;
    // (the run is the point's every observation; meaningful at the run's last lane)
    const bool whole = (__shfl(first ? 1 : 0, head, 64) != 0) && last;
    const double* Mi = d.mp + 9 * (size_t)jj;
    double M[9];
    for (int c = 0; c < 9; ++c) M[c] = Mi[c];
    const double* vk = v + 15 * (size_t)k;
    double W[18];
    load_w<WT>(d.wp, i, W);
    double t[3];
    for (int c = 0; c < 3; ++c) {
        double u = 0.0;
        for (int a = 0; a < 6; ++a) u += W[3 * a + c] * vk[a];
        t[c] = seg.sum(valid ? u : 0.0);
    }
    double tz = 0.0, o[3] = {0.0, 0.0, 0.0};
    if (valid && l == end) {
        if (whole) {
            if (add)
                for (int c = 0; c < 3; ++c) t[c] += add[3 * (size_t)j + c];
            for (int a = 0; a < 3; ++a) {
                o[a] = sign * (M[3 * a] * t[0] + M[3 * a + 1] * t[1] + M[3 * a + 2] * t[2]);
                z[3 * (size_t)j + a] = o[a];
                tz += t[a] * o[a];
            }
        } else {
            for (int a = 0; a < 3; ++a) atomic_add(d.tb + 3 * (size_t)j + a, t[a]);
        }
    }
    if (kFuse) {
        // the least keyframe of the workgroup's observations
        int km = valid ? k : 0x7fffffff;
        for (int off = 32; off > 0; off >>= 1) km = min(km, __shfl_xor(km, off, 64));
        if (l == 0) kmin_w[threadIdx.x >> 6] = km;
        for (int e = threadIdx.x; e < kKfWin * 6; e += blockDim.x) part[e] = 0.0;
        __syncthreads();
        int kbase = 0x7fffffff;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) kbase = min(kbase, kmin_w[w]);
        // z_j and the run's wholeness from its last lane (`whole` holds
        // there only)
        double zj[3];
        for (int a = 0; a < 3; ++a) zj[a] = __shfl(o[a], end, 64);
        const bool run_whole = __shfl(whole ? 1 : 0, end, 64) != 0;
        if (valid && run_whole) {
            const int kk = k - kbase;
            for (int a = 0; a < 6; ++a) {
                const double y = W[3 * a] * zj[0] + W[3 * a + 1] * zj[1] + W[3 * a + 2] * zj[2];
                if (kk < kKfWin) atomicAdd(part + 6 * kk + a, -y);
                else if (k != 0) atomic_add(q + 15 * (size_t)k + a, -y);
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; kbase != 0x7fffffff && e < kKfWin * 6; e += blockDim.x) {
            const int kf = kbase + e / 6;
            const double val = part[e];
            if (val != 0.0 && kf < d.K && kf != 0) atomic_add(q + 15 * (size_t)kf + e % 6, val);
        }
    }
    if (acc) {
        tz = block_sum_vi(tz, red);
        if (threadIdx.x == 0) atomic_add(acc + blockIdx.x % kPqParts, -tz);
    }
}

// the keyframe side of the product for the observations of split points:
// q_k -= W_e z_j, one lane per such observation (their slots in lslot)
template <typename WT>
__global__ void k_vi_long_kf(VIDev d, const double* __restrict__ z, double* __restrict__ q,
                             const double* __restrict__ ps) {
    if (pcg_done(ps)) return;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= d.nlslot) return;
    const long long i = d.lslot[t];
    const int j = d.qpt[i], k = d.qkf[i];
    if (k == 0) return;
    double W[18];
    load_w<WT>(d.wp, i, W);
    const double zj[3] = {z[3 * (size_t)j], z[3 * (size_t)j + 1], z[3 * (size_t)j + 2]};
    for (int a = 0; a < 6; ++a)
        atomic_add(q + 15 * (size_t)k + a, -(W[3 * a] * zj[0] + W[3 * a + 1] * zj[1] + W[3 * a + 2] * zj[2]));
}

// the points split across wavefronts (more than 64 observations): z_j =
// sign C_j^-1 (t_j + add_j) from the parts in tb, -t_j . z_j into acc, tb
// cleared for the next pass; one lane per such point
__global__ void k_vi_long_pts(VIDev d, const double* __restrict__ add, double sign, double* __restrict__ z,
                              const double* __restrict__ ps, double* __restrict__ acc) {
    if (pcg_done(ps)) return;
    __shared__ double red[16];
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    double tz = 0.0;
    if (q < d.nlong) {
        const int j = d.longp[q];
        double t[3];
        for (int c = 0; c < 3; ++c) {
            t[c] = d.tb[3 * (size_t)j + c] + (add ? add[3 * (size_t)j + c] : 0.0);
            d.tb[3 * (size_t)j + c] = 0.0;
        }
        const double* Mi = d.mp + 9 * (size_t)j;
        for (int a = 0; a < 3; ++a) {
            const double o = sign * (Mi[3 * a] * t[0] + Mi[3 * a + 1] * t[1] + Mi[3 * a + 2] * t[2]);
            z[3 * (size_t)j + a] = o;
            tz += t[a] * o;
        }
    }
    if (acc) {
        tz = block_sum_vi(tz, red);
        if (threadIdx.x == 0) atomic_add(acc + blockIdx.x % kPqParts, -tz);
    }
}

// sm_k = sum_{e of k} W_e C_j^-1 W_e^T (the pose block's Schur term for the
// preconditioner: the diagonal block of S when each keyframe sees a point at
// most once), and r_k -= sum_{e of k} W_e z_j(e): observations in keyframe
// order, summed across the keyframe's run of the wavefront
template <typename WT>
__global__ void k_vi_schur_blocks(VIDev d, const double* __restrict__ z, double* __restrict__ r) {
    const long long e0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const bool valid = e0 < d.M;
    const long long e = valid ? e0 : d.M - 1;
    const int k = d.kf[e], j = d.pt[e];
    const int l = (int)(threadIdx.x & 63);
    const int kprev = __shfl_up(k, 1, 64);
    const bool start = !valid || l == 0 || kprev != k;
    const SegScan seg(start);
    int head, end;
    segment_of(__ballot(start), l, head, end);
    const double* Mi = d.mp + 9 * (size_t)j;
    double W[6][3], G[6][3], Wf[18];
    load_w<WT>(d.wk, e, Wf);
    for (int a = 0; a < 6; ++a)
        for (int c = 0; c < 3; ++c) W[a][c] = valid ? Wf[3 * a + c] : 0.0;
    for (int a = 0; a < 6; ++a)
        for (int c = 0; c < 3; ++c) G[a][c] = W[a][0] * Mi[c] + W[a][1] * Mi[3 + c] + W[a][2] * Mi[6 + c];
    const bool out = valid && l == end && k != 0;
    double* S = d.sm + 36 * (size_t)k;
    const double zj[3] = {z[3 * (size_t)j], z[3 * (size_t)j + 1], z[3 * (size_t)j + 2]};
    for (int a = 0; a < 6; ++a) {
        const double y = seg.sum(W[a][0] * zj[0] + W[a][1] * zj[1] + W[a][2] * zj[2]);
        if (out) atomic_add(r + 15 * (size_t)k + a, -y);
    }
    for (int a = 0; a < 6; ++a)
        for (int c = a; c < 6; ++c) {
            const double h = seg.sum(G[a][0] * W[c][0] + G[a][1] * W[c][1] + G[a][2] * W[c][2]);
            if (out) {
                atomic_add(S + 6 * a + c, h);
                if (c != a) atomic_add(S + 6 * c + a, h);
            }
        }
}

// ---- the visual blocks of S explicitly.  S's keyframe-keyframe blocks from
// the points are sparse on a trajectory (a point is seen by a few keyframes
// near each other): 2,000 keyframes with 2.07M observations have 24k blocks of
// 6 x 6 (7 MB), where an implicit product streams W and its indices (212 MB, 43 us).
// They are formed once per step from the same stored W and C^-1 in FP64, and an
// iteration reads them from the L2.

// The run of a point-order slot (its point's other observations) as [lo, hi)
__device__ __forceinline__ void vi_run(const VIDev& d, int q, int& lo, int& hi) {
    const int j = d.qpt[q];
    lo = q;
    while (lo > 0 && d.qpt[lo - 1] == j) --lo;
    hi = q + 1;
    while (hi < d.Mp && d.qpt[hi] == j) ++hi;
}

// One workgroup per keyframe: its covisible keyframes counted in LDS (hist,
// K ints).  kFill = false: the number of blocks and of pairs with later
// keyframes; true (after the scan): the columns, the blocks' first pairs and
// the pairs.
template <bool kFill>
__global__ __launch_bounds__(256) void k_vi_pattern(VIDev d) {
    extern __shared__ int hist[];
    __shared__ int wsum[2][4];
    const int k = blockIdx.x, tid = (int)threadIdx.x;
    for (int c = tid; c < d.K; c += 256) hist[c] = 0;
    __syncthreads();
    for (int e = d.kfoff[k] + tid; e < d.kfoff[k + 1]; e += 256) {
        const int q = d.kslot[e];
        int lo, hi;
        vi_run(d, q, lo, hi);
        for (int u = lo; u < hi; ++u)
            if (u != q) atomicAdd(&hist[d.qkf[u]], 1);
    }
    __syncthreads();
    // running counts over the columns, 256 at a time
    const int l = tid & 63, w = tid >> 6;
    int nb = 0, ni = 0;
    for (int c0 = 0; c0 < d.K; c0 += 256) {
        const int c = c0 + tid;
        const int h = c < d.K ? hist[c] : 0;
        int b = h > 0 ? 1 : 0, it = c > k ? h : 0;
        const int bown = b, iown = it;
        for (int off = 1; off < 64; off <<= 1) {
            const int tb = __shfl_up(b, off, 64), ti = __shfl_up(it, off, 64);
            if (l >= off) {
                b += tb;
                it += ti;
            }
        }
        if (l == 63) {
            wsum[0][w] = b;
            wsum[1][w] = it;
        }
        __syncthreads();
        int pb = nb, pi = ni;
        for (int v = 0; v < 4; ++v) {
            if (v < w) {
                pb += wsum[0][v];
                pi += wsum[1][v];
            }
            nb += wsum[0][v];
            ni += wsum[1][v];
        }
        if (kFill && bown) {
            const int at = d.nrow[k] + pb + b - 1;
            const int first = d.nitem[k] + pi + it - iown;
            d.ncol[at] = c;
            d.nkf[at] = k;
            d.noff[at] = first;
            hist[c] = first;   // the cursor of the fill
        }
        __syncthreads();
    }
    if (!kFill) {
        if (tid == 0) {
            d.nrow[k] = nb;
            d.nitem[k] = ni;
        }
        return;
    }
    // the pairs, by one wavefront in keyframe order (64 observations at a
    // time, a partner each), so that a block's pairs ascend in both
    // observations: lanes of one block are ranked by ballots
    if (w > 0) return;
    for (int e = d.kfoff[k] + l; e - l < d.kfoff[k + 1]; e += 64) {
        const bool in = e < d.kfoff[k + 1];
        const int q = in ? d.kslot[e] : 0, j = in ? d.qpt[q] : -2;
        for (int u = q + 1; ; ++u) {   // a run is in keyframe order
            const bool pair = in && u < d.Mp && d.qpt[u] == j;
            uint64_t left = __ballot(pair);
            if (!left) break;
            const int c = pair ? d.qkf[u] : -1;
            while (left) {
                const int lead = __ffsll((long long)left) - 1;
                const int m = __builtin_amdgcn_readlane(c, lead);
                const uint64_t same = __ballot(c == m);
                if (c == m) d.items[hist[m] + __popcll(same & ((1ull << l) - 1ull))] = make_int2(e, d.kinv[u]);
                __builtin_amdgcn_wave_barrier();
                if (l == lead) hist[m] += __popcll(same);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                left &= ~same;
            }
        }
    }
}

// counts -> offsets of both arrays (exclusive, the totals last), one workgroup
__global__ __launch_bounds__(1024) void k_vi_pattern_scan(VIDev d) {
    __shared__ int wsum[2][16];
    const int tid = (int)threadIdx.x, l = tid & 63, w = tid >> 6;
    int nb = 0, ni = 0;
    for (int k0 = 0; k0 < d.K; k0 += 1024) {
        const int k = k0 + tid;
        int b = k < d.K ? d.nrow[k] : 0, it = k < d.K ? d.nitem[k] : 0;
        const int bown = b, iown = it;
        for (int off = 1; off < 64; off <<= 1) {
            const int tb = __shfl_up(b, off, 64), ti = __shfl_up(it, off, 64);
            if (l >= off) {
                b += tb;
                it += ti;
            }
        }
        if (l == 63) {
            wsum[0][w] = b;
            wsum[1][w] = it;
        }
        __syncthreads();
        int pb = nb, pi = ni;
        for (int v = 0; v < 16; ++v) {
            if (v < w) {
                pb += wsum[0][v];
                pi += wsum[1][v];
            }
            nb += wsum[0][v];
            ni += wsum[1][v];
        }
        if (k < d.K) {
            d.nrow[k] = pb + b - bown;
            d.nitem[k] = pi + it - iown;
        }
        __syncthreads();
    }
    if (tid == 0) {
        d.nrow[d.K] = nb;
        d.nrow[d.K + 1] = 0;
        d.nitem[d.K] = ni;
    }
}

// The observations outside their workgroup's window of keyframes in the
// implicit product (k_vi_schur_pts adds those to q one by one), into
// nrow[K + 1].
__global__ __launch_bounds__(kFuseBlock) void k_vi_far(VIDev d) {
    __shared__ int kmin_w[kFuseBlock / 64];
    const long long i = blockIdx.x * (long long)kFuseBlock + threadIdx.x;
    const bool valid = i < d.Mp && d.qpt[i] >= 0;
    const int k = valid ? d.qkf[i] : 0x7fffffff;
    int km = k;
    for (int off = 32; off > 0; off >>= 1) km = min(km, __shfl_xor(km, off, 64));
    if ((threadIdx.x & 63) == 0) kmin_w[threadIdx.x >> 6] = km;
    __syncthreads();
    for (int w = 0; w < kFuseBlock / 64; ++w) km = min(km, kmin_w[w]);
    const uint64_t far = __ballot(valid && k - km >= kKfWin);
    if ((threadIdx.x & 63) == 0 && far) atomicAdd(d.nrow + d.K + 1, __popcll(far));
}

// V_kk' = -sum W_a C^-1 W_b^T over the block's pairs, stored at (k, k') and,
// transposed, at (k', k).  kWaves wavefronts share a block's pairs (four
// where few blocks would leave the chip idle).  Bound by the reads of W in
// keyframe order, where a block's observations on both sides ascend together
// (in point order the same reads took a line for each lane: 634 us a step at
// 2,000 keyframes).
template <typename WT, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void k_vi_form_blocks(VIDev d) {
    __shared__ double red[kWaves][64];
    const int i = blockIdx.x, k = d.nkf[i], kk = d.ncol[i];
    if (kk <= k) return;
    const int l = lane_id(), w = (int)threadIdx.x >> 6;
    const int last = i + 1 < d.nrow[k + 1] ? d.noff[i + 1] : d.nitem[k + 1];
    double acc[36];
#pragma unroll
    for (int u = 0; u < 36; ++u) acc[u] = 0.0;
    for (int t = d.noff[i] + (int)threadIdx.x; t < last; t += 64 * kWaves) {
        const int2 it = d.items[t];
        const double* Mi = d.mp + 9 * (size_t)d.pt[it.x];
        double A[18], B[18], M[9];
        load_w<WT>(d.wk, it.x, A);
        load_w<WT>(d.wk, it.y, B);
#pragma unroll
        for (int c = 0; c < 9; ++c) M[c] = Mi[c];
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            const double g0 = A[3 * a] * M[0] + A[3 * a + 1] * M[3] + A[3 * a + 2] * M[6];
            const double g1 = A[3 * a] * M[1] + A[3 * a + 1] * M[4] + A[3 * a + 2] * M[7];
            const double g2 = A[3 * a] * M[2] + A[3 * a + 1] * M[5] + A[3 * a + 2] * M[8];
#pragma unroll
            for (int b = 0; b < 6; ++b) acc[6 * a + b] += g0 * B[3 * b] + g1 * B[3 * b + 1] + g2 * B[3 * b + 2];
        }
    }
    wave_sum_scatter(acc);   // sum u in lane rev6(u)
    red[w][rev6(l)] = acc[0];
    __syncthreads();
    const int u = (int)threadIdx.x;
    if (u >= 36) return;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v -= red[q][u];
    d.vblk[36 * (size_t)i + u] = v;
    // the transposed block's place in row k' (its columns ascend)
    int lo = d.nrow[kk], hi = d.nrow[kk + 1] - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (d.ncol[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    d.vblk[36 * (size_t)lo + 6 * (u % 6) + u / 6] = v;
}

// S p for the 15 rows of a keyframe by one wavefront.  The lanes are used
// twice: rows of 16 lanes take the diagonal block and the two cross blocks
// (lane 16 part + row, part 0..2; columns of ad, cbt and cb, so consecutive
// lanes read consecutive entries), and eights of lanes the visual blocks'
// rows (lane 8 s + r, r < 6, of eight neighbours at a time).  Both are summed
// across the lanes without LDS; lane r < 15 returns row r.
__device__ __forceinline__ const double* vi_s_block(const VIDev& d, int k, int part, int& kk) {
    kk = part == 0 ? k : part == 1 ? k + 1 : part == 2 ? k - 1 : -1;
    if (kk < 0 || kk >= d.K) {
        kk = -1;
        return d.ad;
    }
    return part == 0 ? d.ad + 225 * (size_t)k : part == 1 ? d.cbt + 225 * (size_t)k : d.cb + 225 * (size_t)(k - 1);
}

__device__ __forceinline__ double vi_s_total(double u, double v) {
    // u: the parts' rows (lanes 16 apart); v: the neighbours' rows (8 apart)
    u = swap_add<16>(u, u);
    u = swap_add<32>(u, u);
    v += SegScan::move<0x128, 0xF>(v);
    v = swap_add<16>(v, v);
    v = swap_add<32>(v, v);
    return u + (lane_id() < 6 ? v : 0.0);
}

// The row's operands that do not depend on the decision (requested before it):
// the dense blocks, the parts' entries of z and p_old (one lane each), and the
// first eight neighbours' blocks and entries.
struct VISRow {
    double m[15], za, pa, zn, pn;
    double2 b0, b1, b2;
    int n0, n1;
    __device__ __forceinline__ void neighbour(const VIDev& d, const double* __restrict__ z,
                                              const double* __restrict__ p_old, int i0) {
        const int s = lane_id() >> 3, r = lane_id() & 7;
        const bool nb = i0 + s < n1 && r < 6;
        const int i = nb ? i0 + s : n0;
        zn = pn = 0.0;
        if (n0 < n1) {   // uniform
            const double2* B = (const double2*)(d.vblk + 36 * (size_t)i + 6 * min(r, 5));
            b0 = B[0];
            b1 = B[1];
            b2 = B[2];
            const size_t e = 15 * (size_t)d.ncol[i] + min(r, 5);
            zn = nb ? z[e] : 0.0;
            pn = nb ? p_old[e] : 0.0;
        }
    }
    __device__ __forceinline__ void load(const VIDev& d, int k, const double* __restrict__ z,
                                         const double* __restrict__ p_old) {
        const int l = lane_id(), part = l >> 4, row = l & 15;
        n0 = d.nrow[k];
        n1 = d.nrow[k + 1];
        int kk;
        const double* M = vi_s_block(d, k, part, kk);
#pragma unroll
        for (int c = 0; c < 15; ++c) m[c] = M[15 * c + min(row, 14)];
        const bool in = kk >= 0 && row < 15;
        za = in ? z[15 * (size_t)kk + row] : 0.0;
        pa = in ? p_old[15 * (size_t)kk + row] : 0.0;
        neighbour(d, z, p_old, n0);
    }
    // row r < 15 of S (z + beta p_old) in lane r; buf: 128 doubles of LDS of
    // this wavefront
    __device__ __forceinline__ double product(const VIDev& d, const double* __restrict__ z,
                                              const double* __restrict__ p_old, double beta, double* buf) {
        const int l = lane_id(), part = l >> 4, s = l >> 3, r = l & 7;
        buf[l] = za + beta * pa;
        double v = 0.0;
        for (int i0 = n0; i0 < n1; i0 += 8) {   // uniform
            if (i0 > n0) neighbour(d, z, p_old, i0);
            __builtin_amdgcn_wave_barrier();
            buf[64 + l] = zn + beta * pn;
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const double* ps = buf + 64 + 8 * s;
            const double t = b0.x * ps[0] + b0.y * ps[1] + b1.x * ps[2] + b1.y * ps[3] + b2.x * ps[4] + b2.y * ps[5];
            v += i0 + s < n1 && r < 6 ? t : 0.0;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        double u = 0.0;
        const double* ps = buf + 16 * part;
#pragma unroll
        for (int c = 0; c < 15; ++c) u += m[c] * ps[c];
        return vi_s_total(u, v);
    }
};

// The decisions about the PCG step before this one (k_vi_pcg_dir's rules, from
// slot prev_slot), taken alike by every workgroup and recorded by `lead`:
// false when the PCG ends; save and restore act on the caller's own entries.
template <typename Save, typename Restore>
__device__ __forceinline__ bool vi_pcg_go_on(double* __restrict__ ps, int prev_slot, bool lead, double* red,
                                             double* sums, const Save& save, const Restore& restore,
                                             double& beta) {
    double* acc = ps + kAccN * prev_slot;
    const double* prev = ps + kAccN * ((prev_slot + kSlots - 1) % kSlots);
    const double a = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccRrP + threadIdx.x] : 0.0, red);
    __syncthreads();
    const double b = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccRzP + threadIdx.x] : 0.0, red);
    if (threadIdx.x == 0) {
        sums[0] = a;
        sums[1] = b;
    }
    __syncthreads();
    const double rr = sums[0], least = prev[kAccMin], ratio2 = ps[kRatio2];
    double nmin = least;
    bool stop = acc[kAccBreak] != 0.0;
    if (!stop && ratio2 > 0.0) {
        if (rr < least) {
            nmin = rr;
            save();
        } else if (rr > ratio2 * least) {
            restore();
            stop = true;
        }
    }
    if (!stop && rr <= ps[kThr]) stop = true;
    if (lead) {
        acc[kAccRr] = rr;
        acc[kAccRz] = sums[1];
        acc[kAccMin] = nmin;
        if (stop) acc[kAccStop] = 1.0;   // the update kernel sets the stop flag from it
    }
    beta = sums[1] / prev[kAccRz];
    return !stop;
}

// One PCG step in two launches.  First: the decisions about the step before
// (k_vi_pcg_dir's, from slot `prev_slot`; none at the first step), the
// direction p = z + beta p_old formed as it is read (p_old and the new p are
// separate buffers), q = S p and p.q into slot `slot`; one wavefront per
// keyframe.  last: only the decisions about the last step.
// At 2,000 keyframes it takes 9.4 us and the update 5.2 us, where the
// three kernels around the implicit product took 60 (the solve from 87 to 21 ms).
__global__ __launch_bounds__(256) void k_vi_s_prod(VIDev d, double* __restrict__ ps, int slot,
                                                  int prev_slot, int first, int last,
                                                  const double* __restrict__ z,
                                                  const double* __restrict__ p_old, double* __restrict__ p_new,
                                                  double* __restrict__ q, double* __restrict__ x,
                                                  double* __restrict__ xb) {
    __shared__ double red[16];
    __shared__ double sums[2];
    __shared__ double buf[4][128];
    const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k = (int)blockIdx.x * 4 + w;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const size_t own = 15 * (size_t)k + l;
    const bool mine = k < d.K && l < 15;
    // (the rows are requested before the decision's two dependent sums)
    VISRow rows;
    double zo = 0.0, po = 0.0;
    if (k < d.K && !last) {
        rows.load(d, k, z, p_old);
        zo = mine ? z[own] : 0.0;
        po = mine ? p_old[own] : 0.0;
    }
    if (ps[kDone] != 0.0) return;   // set by the update kernel only
    double beta = 0.0;
    if (!first) {
        const bool go = vi_pcg_go_on(ps, prev_slot, lead, red, sums, [&] { if (mine) xb[own] = x[own]; },
                                     [&] { if (mine) x[own] = xb[own]; }, beta);
        if (!go || last) return;
    }
    double pq = 0.0;
    if (k < d.K) {   // whole wavefronts
        const double qv = rows.product(d, z, p_old, beta, buf[w]);
        if (mine) {
            const double pv = zo + beta * po;
            p_new[own] = pv;
            q[own] = qv;
            pq = pv * qv;
        }
    }
    pq = block_sum_vi(pq, red);
    if (threadIdx.x == 0) atomic_add(ps + kAccN * slot + kAccPq + blockIdx.x % kPqParts, pq);
}

// Second: alpha, x, r, z = M^-1 r and the parts of r.r and r.z (as
// k_vi_pcg_update); the stop decided by the first kernel becomes the stop
// flag, and the next step's slot is cleared (no kernel in flight reads it).
// full (the whole-system form): the points are unknowns too (three lanes per
// point in the workgroups after the keyframe ones), and q is cleared for the
// next product.
constexpr int kUpdPts = 85;   // points per 256-lane workgroup of the update
__global__ __launch_bounds__(256) void k_vi_s_update(VIDev d, int full, double* __restrict__ ps, int slot,
                                                    int prev_slot, const double* __restrict__ p,
                                                    double* __restrict__ q, double* __restrict__ x,
                                                    double* __restrict__ r, double* __restrict__ z) {
    __shared__ double rs[256];
    __shared__ double red[16];
    __shared__ double pq_s;
    const long long kf_blocks = (d.K + 15) / 16;
    const bool pts = blockIdx.x >= kf_blocks;
    const int t = (int)threadIdx.x, sub = pts ? t / 3 : t >> 4, row = pts ? t - 3 * sub : t & 15;
    const long long k = pts ? (blockIdx.x - kf_blocks) * (long long)kUpdPts + sub : blockIdx.x * 16LL + sub;
    const bool act = pts ? sub < kUpdPts && k < d.N : k < d.K && row < 15;
    const size_t i = pts ? 15 * (size_t)d.K + 3 * (size_t)k + row : 15 * (size_t)k + row;
    // (requested before the sum of p.q)
    double xi = 0.0, pi = 0.0, qi = 0.0, ri = 0.0, m[15];
    if (act) {
        xi = x[i];
        pi = p[i];
        qi = q[i];
        ri = r[i];
        const double* M = pts ? d.mp + 9 * (size_t)k + 3 * row : d.mki + 225 * (size_t)k + 15 * row;
#pragma unroll
        for (int c = 0; c < 15; ++c) m[c] = c < 3 || !pts ? M[c] : 0.0;
    }
    if (ps[kDone] != 0.0) return;
    double* acc = ps + kAccN * slot;
    if (ps[kAccN * prev_slot + kAccStop] != 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) ps[kDone] = 1.0;
        return;
    }
    if (blockIdx.x == 0)
        for (int e = threadIdx.x; e < kAccN; e += blockDim.x) ps[kAccN * ((slot + 1) % kSlots) + e] = 0.0;
    const double part = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccPq + threadIdx.x] : 0.0, red);
    if (threadIdx.x == 0) pq_s = part;
    __syncthreads();
    const double pq = pq_s;
    if (!(pq > 0.0)) {   // breakdown: decided by every workgroup alike
        if (blockIdx.x == 0 && threadIdx.x == 0) acc[kAccBreak] = 1.0;
        return;
    }
    const double alpha = ps[kAccN * prev_slot + kAccRz] / pq;
    double rr = 0.0, rz = 0.0, rn = 0.0;
    if (act) {
        x[i] = xi + alpha * pi;
        rn = ri - alpha * qi;
        r[i] = rn;
        if (full) q[i] = 0.0;
    }
    rs[threadIdx.x] = rn;
    __syncthreads();
    if (act) {
        double u = 0.0;
        const double* rk = rs + (pts ? 3 : 16) * sub;
        if (pts) {
            u = m[0] * rk[0] + m[1] * rk[1] + m[2] * rk[2];
        } else {
#pragma unroll
            for (int c = 0; c < 15; ++c) u += m[c] * rk[c];
        }
        z[i] = u;
        rr = rn * rn;
        rz = rn * u;
    }
    rr = block_sum_vi(rr, red);
    __syncthreads();
    rz = block_sum_vi(rz, red);
    if (threadIdx.x == 0) {
        atomic_add(acc + kAccRrP + blockIdx.x % kPqParts, rr);
        atomic_add(acc + kAccRzP + blockIdx.x % kPqParts, rz);
        if (blockIdx.x == 0) ps[kSteps] += 1.0;
    }
}

// The whole-system form's PCG step in two launches, this one and the update
// above: the decisions about the step before and the direction p = z + beta
// p_old as in k_vi_s_prod, then q = (H + lambda D) p (q is zero on entry) and
// p.q.  Workgroups over the padded point-order observations, then over the
// inertial terms, then over the rows (p itself and the damping).
//
// An observation's Jacobian is (P [Xc]x, -P R^T | P R^T), so with w = Xc x'
// v_theta + R^T (v_X - v_p) its part of H p is u = P w, g = P^T u and R g, -R
// g, [Xc]x^T g: 32 bytes an observation (Xc and the whitening factor) in
// place of the 216 of a stored Jacobian, and fewer operations.  The keyframes
// of a workgroup lie close together (points are numbered by first observing
// keyframe): those of a window of kKfWin keep rotation, direction and partial
// sums in LDS, one further out goes through memory.  The point rows are
// summed across the point's run of the wavefront and stored by its last lane
// (parts of a point split across wavefronts are added).
//
// quad: only v.H v into the parts of quad (v in z; lambda 0).
//
// At 300 keyframes and 0.31M observations it takes 15.7 us, the update 7.0,
// where the stored Jacobian's product (18.9), the inertial product (6.8), the
// damping, dot and direction kernels (12.2) and the update took 45.
enum { kFullFirst = 0, kFullNext, kFullLast, kFullQuad };
__global__ __launch_bounds__(kFuseBlock) void k_vi_full_prod(VIDev d, double lam, double* __restrict__ ps, int slot,
                                                            int prev_slot, int mode, const double* __restrict__ z,
                                                            const double* __restrict__ p_old,
                                                            double* __restrict__ p_new, double* __restrict__ q,
                                                            double* __restrict__ x, double* __restrict__ xb,
                                                            double* __restrict__ quad) {
    __shared__ double red[16];
    __shared__ double sums[2];
    __shared__ double part[kKfWin * 6];
    __shared__ double win[kKfWin * 15];   // direction (6) and rotation (9)
    __shared__ int kmin_w[16];
    const bool only_quad = mode == kFullQuad;
    if (!only_quad && ps[kDone] != 0.0) return;   // set by the update kernel only
    const long long n = 15LL * d.K + 3 * d.N, st_blocks = (d.Mp + kFuseBlock - 1) / kFuseBlock, in_blocks = (d.K + 6) / 8;
    const int tid = (int)threadIdx.x, l = tid & 63;
    const long long rb = blockIdx.x - st_blocks - in_blocks;
    const size_t own = (size_t)(rb * kFuseBlock + tid);
    const bool mine = rb >= 0 && (long long)own < n;
    const bool next = mode == kFullNext;
    double beta = 0.0;
    if (next || mode == kFullLast) {
        const bool go = vi_pcg_go_on(ps, prev_slot, blockIdx.x == 0 && tid == 0, red, sums,
                                     [&] { if (mine) xb[own] = x[own]; }, [&] { if (mine) x[own] = xb[own]; }, beta);
        if (!go || !next) return;
    }
    auto p = [&](size_t i) { return next ? z[i] + beta * p_old[i] : z[i]; };
    double pq = 0.0;
    if (blockIdx.x < st_blocks) {
        const long long i = blockIdx.x * (long long)kFuseBlock + tid < d.Mp
                                ? blockIdx.x * (long long)kFuseBlock + tid : d.Mp - 1;
        const int jq = d.qpt[i];
        const bool valid = blockIdx.x * (long long)kFuseBlock + tid < d.Mp && jq >= 0;
        const int j = valid ? jq : 0, k = valid ? d.qkf[i] : 0;
        const size_t op = 15 * (size_t)d.K + 3 * (size_t)j;
        double jc[4], vx[3];
        js_load(d, i, jc);
        for (int c = 0; c < 3; ++c) vx[c] = p(op + c);
        const int jprev = __shfl_up(jq, 1, 64);
        const bool start = !valid || l == 0 || jprev != jq;
        const SegScan seg(start);
        int head, end;
        segment_of(__ballot(start), l, head, end);
        const bool first = i == 0 || d.qpt[i - 1] != jq;
        const bool lastp = i == d.Mp - 1 || d.qpt[i + 1] != jq;
        const bool has_first = __shfl(first ? 1 : 0, head, 64) != 0;
        const bool whole = has_first && lastp;   // at the run's last lane
        int km = valid ? k : 0x7fffffff;
        for (int off = 32; off > 0; off >>= 1) km = min(km, __shfl_xor(km, off, 64));
        if (l == 0) kmin_w[tid >> 6] = km;
        __syncthreads();
        int kbase = 0x7fffffff;
        for (int w = 0; w < kFuseBlock / 64; ++w) kbase = min(kbase, kmin_w[w]);
        const bool any = kbase != 0x7fffffff;
        for (int e = tid; e < kKfWin * 15; e += kFuseBlock) {
            const int kf = kbase + e / 15, c = e % 15;   // (no further than K when any)
            if (any && kf < d.K) win[e] = c < 6 ? p(15 * (size_t)kf + c) : d.st[(size_t)kSt * kf + c - 6];
        }
        for (int e = tid; e < kKfWin * 6; e += kFuseBlock) part[e] = 0.0;
        __syncthreads();
        double yx[3] = {0.0, 0.0, 0.0};
        if (valid) {
            const int kk = k - kbase;
            double v[6], R[9];
            if (kk < kKfWin) {
                for (int c = 0; c < 6; ++c) v[c] = win[15 * kk + c];
                for (int c = 0; c < 9; ++c) R[c] = win[15 * kk + 6 + c];
            } else {
                for (int c = 0; c < 6; ++c) v[c] = p(15 * (size_t)k + c);
                for (int c = 0; c < 9; ++c) R[c] = d.st[(size_t)kSt * k + c];
            }
            const double X = jc[0], Y = jc[1], Z = jc[2], sc = jc[3], iz = 1.0 / Z;
            const double e0 = vx[0] - v[3], e1 = vx[1] - v[4], e2 = vx[2] - v[5];
            const double w0 = R[0] * e0 + R[3] * e1 + R[6] * e2 + (Y * v[2] - Z * v[1]);
            const double w1 = R[1] * e0 + R[4] * e1 + R[7] * e2 + (Z * v[0] - X * v[2]);
            const double w2 = R[2] * e0 + R[5] * e1 + R[8] * e2 + (X * v[1] - Y * v[0]);
            const double fx = sc * d.fx * iz, fy = sc * d.fy * iz, xz = X * iz, yz = Y * iz,
                         bz = (X - d.base) * iz;
            const double u0 = fx * (w0 - xz * w2), u1 = fy * (w1 - yz * w2), u2 = fx * (w0 - bz * w2);
            pq = u0 * u0 + u1 * u1 + u2 * u2;
            const double g0 = fx * (u0 + u2), g1 = fy * u1, g2 = -(fx * (xz * u0 + bz * u2) + yz * g1);
            for (int c = 0; c < 3; ++c) yx[c] = R[3 * c] * g0 + R[3 * c + 1] * g1 + R[3 * c + 2] * g2;
            if (k != 0 && !only_quad) {
                const double y[6] = {Z * g1 - Y * g2, X * g2 - Z * g0, Y * g0 - X * g1, -yx[0], -yx[1], -yx[2]};
                for (int c = 0; c < 6; ++c) {
                    if (kk < kKfWin) atomicAdd(part + 6 * kk + c, y[c]);
                    else atomic_add(q + 15 * (size_t)k + c, y[c]);
                }
            }
        }
        if (!only_quad) {
            for (int c = 0; c < 3; ++c) {
                const double sy = seg.sum(yx[c]);
                if (valid && l == end) {
                    const double damp = has_first ? lam * d.dg[op + c] * vx[c] : 0.0;
                    if (whole) q[op + c] = sy + damp;
                    else atomic_add(q + op + c, sy + damp);
                }
            }
            __syncthreads();
            for (int e = tid; any && e < kKfWin * 6; e += kFuseBlock) {
                const int kf = kbase + e / 6;
                const double val = part[e];
                if (val != 0.0 && kf < d.K && kf != 0) atomic_add(q + 15 * (size_t)kf + e % 6, val);
            }
        }
    } else if (rb < 0) {
        // the inertial and bias terms: one wavefront per term; lane c < 24
        // holds column c (keyframe i's 15 entries, then keyframe j's first 9)
        const int f = (int)((blockIdx.x - st_blocks) * (kFuseBlock / 64)) + (tid >> 6);
        if (f < d.K - 1) {   // whole wavefronts
            const size_t oi = 15 * (size_t)f, oj = 15 * (size_t)(f + 1);
            const double* J = d.ji + (size_t)216 * f;
            const double* O = d.info + 81 * (size_t)f;
            const bool col = l < 24;
            const double vc = col ? p(l < 15 ? oi + l : oj + (l - 15)) : 0.0;
            double jc[9], u[9];
            for (int a = 0; a < 9; ++a) jc[a] = col ? J[24 * a + l] : 0.0;
            // u = J v (sums over the 24 columns), w = Omega u, y_c = sum_a J[a][c] w[a]
            for (int a = 0; a < 9; ++a) u[a] = wave_sum(jc[a] * vc);
            double y = 0.0, uw = 0.0;
            for (int a = 0; a < 9; ++a) {
                double w = 0.0;
                for (int b = 0; b < 9; ++b) w += O[9 * a + b] * u[b];
                y += jc[a] * w;
                uw += u[a] * w;
            }
            if (l == 0) pq += uw;
            if (col && !only_quad) atomic_add(q + (l < 15 ? oi + l : oj + (l - 15)), y);
            if (l < 6) {
                const double dt = d.pre[(size_t)kPreStride * f + kDt];
                const double wb = (l < 3 ? d.wg : d.wa) / dt;
                const double diff = p(oj + 9 + l) - (f != 0 ? p(oi + 9 + l) : 0.0);
                pq += wb * diff * diff;
                if (!only_quad) {
                    atomic_add(q + oj + 9 + l, wb * diff);
                    if (f != 0) atomic_add(q + oi + 9 + l, -(wb * diff));
                }
            }
        }
    } else if (mine && !only_quad) {
        const double v = p(own), damp = lam * d.dg[own] * v;
        p_new[own] = v;
        pq = damp * v;
        if (own < 15 * (size_t)d.K) atomic_add(q + own, damp);
    }
    pq = block_sum_vi(pq, red);
    if (tid == 0) atomic_add((only_quad ? quad : ps + kAccN * slot + kAccPq) + blockIdx.x % kPqParts, pq);
}

// The whole PCG of a short trajectory (at most kOneKf keyframes) in one
// workgroup of eight wavefronts: keyframe w + 8 t is wavefront w's t-th.  Its
// diagonal, cross and preconditioner blocks stay in registers (two wavefronts
// per SIMD leave 256 VGPRs), the vectors too (a lane per entry: 16 lanes a
// keyframe), the direction and the visual blocks in LDS (their upper half: at
// most 496 of 288 bytes, read along rows or columns); three barriers an
// iteration.  Rules and arithmetic as the two kernels above; r, z from the
// start kernels, x out.  Bound by the iteration's chain of sums, divisions and
// barriers: 3.2 us at 31 keyframes (reading each pair's block once for both
// rows, or taking the direction by DPP instead of from LDS, left it there); 4.5
// with the visual blocks requested from the L2, 14 as three launches of the
// implicit product (5 steps of 200 iterations: the solve from 19.0 to 5.1 ms).
constexpr int kOneKf = 32;
constexpr int kOneBlock = 512;
__global__ __launch_bounds__(kOneBlock) void k_vi_s_pcg_one(VIDev d, double* __restrict__ ps,
                                                           int max_iters, const double* __restrict__ r_in,
                                                           const double* __restrict__ z_in,
                                                           double* __restrict__ x_out) {
    constexpr int kWaves = kOneBlock / 64, kN = 16 * kOneKf, kPer = kOneKf / kWaves, kPre = 4;
    static_assert(kPer == 4 && 8 * kPre >= kOneKf - 1, "a keyframe per 16 lanes; every neighbour in a group");
    extern __shared__ __align__(16) double blocks[];   // 36 doubles per upper block
    __shared__ __align__(16) double p_s[kN], r_s[kN], q_s[kN];
    __shared__ __align__(16) double red[3][kWaves];
    __shared__ int low_s[kOneKf];   // lower blocks in the rows up to this one
    const int l = lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int part = l >> 4, row = l & 15, s = l >> 3, r8 = l & 7;
    const double* a = ps + kAccN * (kSlots - 1);
    double rz = a[kAccRz], rr = a[kAccRr], least = rr;
    const double thr = ps[kThr], ratio2 = ps[kRatio2];
    auto yes = [](bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; };
    const bool idle = yes(ps[kDone] != 0.0);
    // first index in [lo, hi) of a row's ascending columns that is >= c
    auto lower = [&](int lo, int hi, int c) {
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (d.ncol[mid] < c) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    if (w == 0) {
        int c = l < d.K ? lower(d.nrow[l], d.nrow[l + 1], l) - d.nrow[l] : 0;
        for (int off = 1; off < kOneKf; off <<= 1) {
            const int t = __shfl_up(c, off, 64);
            if (l >= off) c += t;
        }
        if (l < kOneKf) low_s[l] = c;
    }
    __syncthreads();
    for (int i = w; i < d.nnz; i += kWaves) {   // uniform
        const int k = d.nkf[i];
        if (d.ncol[i] > k && l < 36) blocks[36 * (i - low_s[k]) + l] = d.vblk[36 * (size_t)i + l];
    }
    // lane 16 t + c owns entry c of the wavefront's keyframe t
    const int k_own = w + kWaves * part, i_own = 16 * k_own + row;
    const bool mine = k_own < d.K && row < 15;
    double x = 0.0, xb = 0.0, z = mine ? z_in[15 * k_own + row] : 0.0, r = mine ? r_in[15 * k_own + row] : 0.0;
    double p = z;
    r_s[i_own] = r;
    p_s[i_own] = p;
    double m[kPer][15], mi[15];
#pragma unroll
    for (int c = 0; c < 15; ++c)   // symmetric: read by columns
        mi[c] = mine ? d.mki[225 * (size_t)k_own + 15 * c + row] : 0.0;
    // nb: a neighbour's block (entry 36 u + r8 or 6 r8 of blocks), whether it
    // is read by columns, and its keyframe
    int pb[kPer], nn[kPer], nb[kPer][kPre];
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        const int k = w + kWaves * t;
        const bool on = k < d.K;
        int kk = -1;
        const double* M = on ? vi_s_block(d, k, part, kk) : d.ad;
        pb[t] = 16 * max(kk, 0);
#pragma unroll
        for (int c = 0; c < 15; ++c) m[t][c] = kk >= 0 && row < 15 ? M[15 * c + min(row, 14)] : 0.0;
        const int n0 = on ? __builtin_amdgcn_readfirstlane(d.nrow[k]) : 0;
        nn[t] = on ? __builtin_amdgcn_readfirstlane(d.nrow[k + 1]) - n0 : 0;
#pragma unroll
        for (int g = 0; g < kPre; ++g) {
            nb[t][g] = -1;
            if (8 * g + s < nn[t] && r8 < 6) {
                const int i = n0 + 8 * g + s, c = d.ncol[i];
                const int u = c > k ? i - low_s[k] : lower(d.nrow[c], d.nrow[c + 1], k) - low_s[c];
                nb[t][g] = (36 * u + (c > k ? 6 * r8 : r8)) << 8 | (c > k ? 0 : 128) | c;
            }
        }
    }
    auto total = [&](int c) {   // the wavefronts' sums
        const double* v = red[c];
        return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    };
    int steps = 0;
    while (!idle && steps < max_iters) {   // uniform: every thread holds the same scalars
        __syncthreads();   // the direction is complete
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            if (w + kWaves * t >= d.K) break;   // uniform
            double v = 0.0;
#pragma unroll
            for (int g = 0; g < kPre; ++g) {
                if (8 * g >= nn[t]) break;   // uniform
                int at = nb[t][g];
                asm volatile("" : "+v"(at));   // its addresses are made here, not kept: registers
                if (at >= 0) {
                    const double* B = blocks + (at >> 8);
                    const double* q6 = p_s + 16 * (at & 31);
                    const int st = (at & 128) ? 6 : 1;
                    double h0 = 0.0, h1 = 0.0;
#pragma unroll
                    for (int c = 0; c < 6; c += 2) {
                        h0 += B[st * c] * q6[c];
                        h1 += B[st * (c + 1)] * q6[c + 1];
                    }
                    v += h0 + h1;
                }
            }
            double u0 = 0.0, u1 = 0.0, u2 = 0.0;
            const double* pk = p_s + pb[t];
#pragma unroll
            for (int c = 0; c < 15; c += 3) {
                u0 += m[t][c] * pk[c];
                u1 += m[t][c + 1] * pk[c + 1];
                u2 += m[t][c + 2] * pk[c + 2];
            }
            const double q = vi_s_total((u0 + u1) + u2, v);
            if (l < 16) q_s[16 * (w + kWaves * t) + l] = q;   // (entry 15 is not used)
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const double q = mine ? q_s[i_own] : 0.0;
        const double pql = wave_sum(p * q);
        if (l == 0) red[0][w] = pql;
        __syncthreads();
        const double pq = total(0);
        if (yes(!(pq > 0.0))) break;   // breakdown: x stays the last iterate
        const double alpha = rz / pq;
        x += alpha * p;
        r -= alpha * q;
        r_s[i_own] = r;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        {
            const double* rk = r_s + 16 * k_own;
            double u0 = 0.0, u1 = 0.0, u2 = 0.0;
#pragma unroll
            for (int c = 0; c < 15; c += 3) {
                u0 += mi[c] * rk[c];
                u1 += mi[c + 1] * rk[c + 1];
                u2 += mi[c + 2] * rk[c + 2];
            }
            z = (u0 + u1) + u2;
        }
        double both = swap_add<32>(r * r, r * z);   // r.r in the low lanes, r.z in the high ones
        both += SegScan::move<0x128, 0xF>(both);
        both += SegScan::move<0x124, 0xF>(both);
        both += SegScan::move<0x122, 0xF>(both);
        both += SegScan::move<0x121, 0xF>(both);
        both = swap_add<16>(both, both);
        if (l == 0) red[1][w] = both;
        if (l == 32) red[2][w] = both;
        __syncthreads();
        rr = total(1);
        const double rz_new = total(2);
        steps += 1;
        if (ratio2 > 0.0) {
            if (yes(rr < least)) {
                least = rr;
                xb = x;
            } else if (yes(rr > ratio2 * least)) {
                x = xb;
                break;
            }
        }
        if (yes(rr <= thr)) break;
        const double beta = rz_new / rz;
        rz = rz_new;
        p = z + beta * p;
        p_s[i_own] = p;
    }
    if (mine) x_out[15 * k_own + row] = x;
    if (threadIdx.x == 0) {
        ps[kSteps] = (double)steps;
        ps[kDone] = 1.0;
    }
}

// the inertial cross blocks of the damped system, once per linearisation:
// icx_f = J_i^T Omega J_j over keyframe i's 15 columns and keyframe j's first
// 9; full: the same as whole 15 x 15 blocks with the bias random walk's
// -Omega_b, and transposed, for the explicit products (one lane per entry)
__global__ void k_vi_cross(VIDev d, int full) {
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= 225LL * (d.K - 1)) return;
    const long long f = t / 225;
    const int a = (int)(t % 225) / 15, c = (int)(t % 15);
    const double* J = d.ji + (size_t)216 * f;
    const double* O = d.info + 81 * (size_t)f;
    double u = 0.0;
    for (int m = 0; m < (c < 9 ? 9 : 0); ++m) {
        double w = 0.0;
        for (int k = 0; k < 9; ++k) w += O[9 * m + k] * J[24 * k + 15 + c];
        u += J[24 * m + a] * w;
    }
    if (c < 9) d.icx[135 * f + 9 * a + c] = u;
    if (!full) return;
    if (a == c && a >= 9 && f != 0) u -= (a < 12 ? d.wg : d.wa) / d.pre[(size_t)kPreStride * f + kDt];
    d.cb[225 * f + 15 * a + c] = u;
    d.cbt[225 * f + 15 * c + a] = u;
}

// the start: threshold tol^2 r0.r0 (r0.r0 and r0.z0 in the last slot, summed
// from their parts by one workgroup of kPqParts);
// nothing to do when r0 is already below it or r0.z0 <= 0.  ratio2: the
// squared rejection ratio (0: no rejection test)
__global__ __launch_bounds__(kPqParts) void k_vi_pcg_init(double* __restrict__ ps, double tol, double ratio2) {
    __shared__ double red[16];
    double* a = ps + kAccN * (kSlots - 1);
    const double rr = block_sum_vi(a[kAccRrP + threadIdx.x], red);
    __syncthreads();
    const double rz = block_sum_vi(a[kAccRzP + threadIdx.x], red);
    if (threadIdx.x != 0) return;
    a[kAccRr] = rr;
    a[kAccRz] = rz;
    const double thr = tol * tol * a[kAccRr];
    ps[kThr] = thr;
    ps[kDone] = (a[kAccRr] > thr && a[kAccRz] > 0.0) ? 0.0 : 1.0;
    ps[kSteps] = 0.0;
    ps[kRatio2] = ratio2;
    a[kAccMin] = a[kAccRr];
    a[kAccStop] = ps[kDone];
}

// step `slot`: alpha = r.z / p.q (a step with p.q <= 0 ends the iteration at
// the current iterate), x += alpha p, r -= alpha q, z = M^-1 r and the new
// r.r, r.z.  16 lanes per keyframe (15 used), the residual block through LDS
// for the 15 x 15 inverse.
__global__ __launch_bounds__(256) void k_vi_pcg_update(VIDev d, double* __restrict__ ps, int slot,
                                                      const double* __restrict__ p,
                                                      const double* __restrict__ q, double* __restrict__ x,
                                                      double* __restrict__ r, double* __restrict__ z) {
    __shared__ double rs[256];
    __shared__ double red[16];
    if (ps[kDone] != 0.0) return;
    double* acc = ps + kAccN * slot;
    __shared__ double pq_s;
    {
        const double part = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccPq + threadIdx.x] : 0.0, red);
        if (threadIdx.x == 0) pq_s = part;
        __syncthreads();
    }
    const double pq = pq_s;
    if (!(pq > 0.0)) {   // breakdown: decided by every workgroup alike
        if (blockIdx.x == 0 && threadIdx.x == 0) acc[kAccBreak] = 1.0;
        return;
    }
    const double alpha = ps[kAccN * ((slot + kSlots - 1) % kSlots) + kAccRz] / pq;
    const long long k = blockIdx.x * 16LL + (threadIdx.x >> 4);
    const int row = (int)(threadIdx.x & 15);
    const bool act = k < d.K && row < 15;
    const size_t i = 15 * (size_t)k + row;
    double rr = 0.0, rz = 0.0, rn = 0.0;
    if (act) {
        x[i] += alpha * p[i];
        rn = r[i] - alpha * q[i];
        r[i] = rn;
    }
    rs[threadIdx.x] = rn;
    __syncthreads();
    if (act) {
        const double* Mi = d.mki + 225 * (size_t)k + 15 * row;
        const double* rk = rs + (threadIdx.x & ~15u);
        double u = 0.0;
        for (int c = 0; c < 15; ++c) u += Mi[c] * rk[c];
        z[i] = u;
        rr = rn * rn;
        rz = rn * u;
    }
    rr = block_sum_vi(rr, red);
    __syncthreads();
    rz = block_sum_vi(rz, red);
    if (threadIdx.x == 0) {
        atomic_add(acc + kAccRrP + blockIdx.x % kPqParts, rr);   // summed by k_vi_pcg_dir
        atomic_add(acc + kAccRzP + blockIdx.x % kPqParts, rz);
        if (blockIdx.x == 0) ps[kSteps] += 1.0;
    }
}

// step `slot`, continued, with the decisions of the PCG rules: a breakdown
// ends at the current iterate; with the rejection test, a new least r.r
// saves x in xb, and r.r > ratio^2 times the least ends the iteration with
// xb restored; r.r <= the threshold ends it; otherwise p = z + beta p with
// beta = r.z / previous r.z.  Every workgroup takes the same decisions from
// this slot's and the previous slot's values (which no workgroup of this
// kernel writes); workgroup 0 records them (this slot's least r.r and stop
// flag, the stop flag the later kernels read) and clears the next slot; qz
// (when given) is cleared for the next product.
__global__ void k_vi_pcg_dir(long long n, double* __restrict__ ps, int slot, const double* __restrict__ z,
                             double* __restrict__ p, double* __restrict__ x, double* __restrict__ xb,
                             double* __restrict__ qz) {
    double* acc = ps + kAccN * slot;
    const double* prev = ps + kAccN * ((slot + kSlots - 1) % kSlots);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const long long st = (long long)gridDim.x * blockDim.x;
    const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    // this step's r.r and r.z from their parts (the same sums, in the same
    // order, in every workgroup); workgroup 0 keeps them in the slot
    __shared__ double red[16];
    __shared__ double sums[2];
    {
        const double a = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccRrP + threadIdx.x] : 0.0, red);
        __syncthreads();
        const double b = block_sum_vi(threadIdx.x < kPqParts ? acc[kAccRzP + threadIdx.x] : 0.0, red);
        if (threadIdx.x == 0) {
            sums[0] = a;
            sums[1] = b;
        }
        __syncthreads();
    }
    if (lead) {
        acc[kAccRr] = sums[0];
        acc[kAccRz] = sums[1];
    }
    if (blockIdx.x == 0)
        for (int e = threadIdx.x; e < kAccN; e += blockDim.x) ps[kAccN * ((slot + 1) % kSlots) + e] = 0.0;
    if (prev[kAccStop] != 0.0 || acc[kAccBreak] != 0.0) {
        if (lead) {
            acc[kAccStop] = 1.0;
            acc[kAccMin] = prev[kAccMin];
            ps[kDone] = 1.0;
        }
        return;
    }
    const double rr = sums[0], least = prev[kAccMin], ratio2 = ps[kRatio2];
    double nmin = least;
    if (ratio2 > 0.0) {
        if (rr < least) {
            nmin = rr;
            for (long long i = i0; i < n; i += st) xb[i] = x[i];
        } else if (rr > ratio2 * least) {
            for (long long i = i0; i < n; i += st) x[i] = xb[i];
            if (lead) {
                acc[kAccStop] = 1.0;
                acc[kAccMin] = least;
                ps[kDone] = 1.0;
            }
            return;
        }
    }
    if (rr <= ps[kThr]) {
        if (lead) {
            acc[kAccStop] = 1.0;
            acc[kAccMin] = nmin;
            ps[kDone] = 1.0;
        }
        return;
    }
    const double beta = sums[1] / prev[kAccRz];
    for (long long i = i0; i < n; i += st) {
        p[i] = z[i] + beta * p[i];
        if (qz) qz[i] = 0.0;   // the next product adds into q
    }
    if (lead) acc[kAccMin] = nmin;
}

// The candidate (R Exp(dtheta), p + dp, v + dv, b + db; X + dX) and the sums
// of a trial that need no other order: |x|^2 of the current state over the
// free parameters, b.dx, |dx|^2 and, in the Schur form, dx_k^T A dx_k +
// sum_j dx_j^T H_pp,j dx_j (undamped) and b_p.dx_p; lanes: keyframes, points,
// then keyframe rows
__global__ __launch_bounds__(256) void k_vi_step(VIDev d, const double* __restrict__ dx, int schur) {
    __shared__ double red[16];
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    double xn = 0.0, bx = 0.0, xx = 0.0, hx = 0.0, bxp = 0.0;
    if (t < d.K) {
        const double* s = d.st + (size_t)kSt * t;
        double* c = d.st_c + (size_t)kSt * t;
        const double* u = dx + 15 * (size_t)t;
        const double w[3] = {u[0], u[1], u[2]};
        double E[3][3];
        so3_exp(w, E);
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
                c[3 * a + b] = s[3 * a] * E[0][b] + s[3 * a + 1] * E[1][b] + s[3 * a + 2] * E[2][b];
        for (int k = 0; k < 12; ++k) c[9 + k] = s[9 + k] + u[3 + k];
        if (t >= 1) {
            double R[3][3], v[3];
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) R[a][b] = s[3 * a + b];
            so3_log(R, v);
            for (int k = 0; k < 3; ++k) xn += v[k] * v[k];
            for (int k = 9; k < kSt; ++k) xn += s[k] * s[k];
        }
    } else if (t < d.K + d.N) {
        const long long j = t - d.K;
        const double* u = dx + 15 * (size_t)d.K + 3 * j;
        const double* b = d.b + 15 * (size_t)d.K + 3 * j;
        for (int k = 0; k < 3; ++k) {
            const double X = d.X[3 * j + k];
            d.X_c[3 * j + k] = X + u[k];
            xn += X * X;
            bxp += b[k] * u[k];
            xx += u[k] * u[k];
        }
        bx = bxp;
        if (schur) {
            const double* H = d.hp + 9 * j;
            for (int a = 0; a < 3; ++a) hx += u[a] * (H[3 * a] * u[0] + H[3 * a + 1] * u[1] + H[3 * a + 2] * u[2]);
        }
    } else if (t < 16LL * d.K + d.N) {
        const long long i = t - d.K - d.N;
        const double u = dx[i];
        bx = d.b[i] * u;
        xx = u * u;
        if (schur) hx = u * vi_ap_row(d, 0.0, dx, i);
    }
    const double sums[kStepSums] = {hx, bxp, bx, xx, xn};
    for (int a = 0; a < kStepSums; ++a) {
        const double v = block_sum_vi(sums[a], red);
        if (threadIdx.x == 0) atomic_add(d.scal + kRedOff + a * kPqParts + blockIdx.x % kPqParts, v);
        __syncthreads();
    }
}

}  // namespace vi
}  // namespace gba

// ------------------------------------------------------------------ C ABI
namespace {

// A recorded run of PCG steps of one solve (its stream is only captured on).
struct StepGraph {
    hipStream_t stream = nullptr;
    hipGraphExec_t exec = nullptr;
    bool failed = false;   // steps are then launched one by one
    StepGraph() = default;
    StepGraph(const StepGraph&) = delete;
    StepGraph& operator=(const StepGraph&) = delete;
    ~StepGraph() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (stream) (void)hipStreamDestroy(stream);
    }
    template <typename Launch>
    bool record(const Launch& launch) {
        hipGraph_t graph = nullptr;
        bool ok = hipStreamCreateWithFlags(&stream, hipStreamNonBlocking) == hipSuccess &&
                  hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
        if (ok) {
            launch(stream);
            ok = hipStreamEndCapture(stream, &graph) == hipSuccess && graph &&
                 hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
        }
        if (graph) (void)hipGraphDestroy(graph);
        if (!ok) {
            exec = nullptr;
            failed = true;
            (void)hipGetLastError();
        }
        return ok;
    }
};

}  // namespace

extern "C" {

gba_status gba_vi_preintegrate(int device, int n, const int64_t* sample_off, const double* gyro,
                               const double* acc, double dt, const double* bias0, double sigma_g,
                               double sigma_a, double* out) {
    if (n < 0 || !sample_off || !bias0 || !out || !(dt > 0.0) || !(sigma_g >= 0.0) || !(sigma_a >= 0.0))
        return GBA_ERR_INVALID_ARG;
    if (n == 0) return GBA_OK;
    for (int f = 0; f < n; ++f)
        if (sample_off[f + 1] < sample_off[f] || sample_off[0] != 0) return GBA_ERR_INVALID_ARG;
    const size_t ns = (size_t)sample_off[n];
    if (ns > 0 && (!gyro || !acc)) return GBA_ERR_INVALID_ARG;
    if (hipSetDevice(device) != hipSuccess) return GBA_ERR_HIP;
    gba::vi::DevBufs b(sizeof(double) * (6 * ns + (gba::vi::kPreStride + 8) * (size_t)n) + 8192);
    long long* doff = nullptr;
    double *dg = nullptr, *da = nullptr, *db = nullptr, *dout = nullptr;
    if (!b.up(&doff, (const long long*)sample_off, (size_t)n + 1) || !b.up(&dg, gyro, 3 * ns) ||
        !b.up(&da, acc, 3 * ns) || !b.up(&db, bias0, 6 * (size_t)n) ||
        !b.up(&dout, (const double*)nullptr, (size_t)gba::vi::kPreStride * n))
        return GBA_ERR_HIP;
    hipLaunchKernelGGL(gba::vi::k_preintegrate, dim3((unsigned)((n + 3LL) / 4)), dim3(64), 0, nullptr, n, doff, dg,
                       da, dt, db, sigma_g, sigma_a, dout);
    if (hipGetLastError() != hipSuccess) return GBA_ERR_HIP;
    if (hipMemcpy(out, dout, sizeof(double) * gba::vi::kPreStride * n, hipMemcpyDeviceToHost) != hipSuccess)
        return GBA_ERR_HIP;
    return GBA_OK;
}

gba_status gba_vi_eval_inertial(int device, int n_kf, const double* states, const double* pre,
                                double* r, double* J) {
    if (n_kf < 0 || (n_kf > 1 && (!states || !pre || !r || !J))) return GBA_ERR_INVALID_ARG;
    const int n = n_kf > 1 ? n_kf - 1 : 0;
    if (n == 0) return GBA_OK;
    if (hipSetDevice(device) != hipSuccess) return GBA_ERR_HIP;
    gba::vi::DevBufs b(sizeof(double) * (15 + gba::vi::kPreStride + 225) * (size_t)n_kf + 8192);
    double *ds = nullptr, *dp = nullptr, *dr = nullptr, *dj = nullptr;
    if (!b.up(&ds, states, 15 * (size_t)n_kf) || !b.up(&dp, pre, (size_t)gba::vi::kPreStride * n) ||
        !b.up(&dr, (const double*)nullptr, 9 * (size_t)n) || !b.up(&dj, (const double*)nullptr, 216 * (size_t)n))
        return GBA_ERR_HIP;
    const long long lanes = 24LL * n;
    hipLaunchKernelGGL(gba::vi::k_inertial_eval, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0,
                       nullptr, n, ds, dp, dr, dj);
    if (hipGetLastError() != hipSuccess) return GBA_ERR_HIP;
    if (hipMemcpy(r, dr, sizeof(double) * 9 * n, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(J, dj, sizeof(double) * 216 * n, hipMemcpyDeviceToHost) != hipSuccess)
        return GBA_ERR_HIP;
    return GBA_OK;
}

gba_status gba_vi_eval_stereo(int device, int n_kf, const double* states, int64_t n_pts,
                              const double* pts, int64_t n_obs, const int64_t* kf, const int64_t* pt,
                              const double* obs, const double* intr, double* r, double* J) {
    if (n_kf < 0 || n_pts < 0 || n_obs < 0 || !intr) return GBA_ERR_INVALID_ARG;
    if (n_obs == 0) return GBA_OK;
    if (!states || !pts || !kf || !pt || !obs || !r || !J) return GBA_ERR_INVALID_ARG;
    for (int64_t e = 0; e < n_obs; ++e)
        if (kf[e] < 0 || kf[e] >= n_kf || pt[e] < 0 || pt[e] >= n_pts) return GBA_ERR_UNKNOWN_ID;
    if (hipSetDevice(device) != hipSuccess) return GBA_ERR_HIP;
    gba::vi::DevBufs b(sizeof(double) * (15 * (size_t)n_kf + 3 * (size_t)n_pts + 35 * (size_t)n_obs) + 8192);
    double *ds = nullptr, *dpts = nullptr, *dobs = nullptr, *dr = nullptr, *dj = nullptr;
    long long *dkf = nullptr, *dpt = nullptr;
    if (!b.up(&ds, states, 15 * (size_t)n_kf) || !b.up(&dpts, pts, 3 * (size_t)n_pts) ||
        !b.up(&dkf, (const long long*)kf, (size_t)n_obs) || !b.up(&dpt, (const long long*)pt, (size_t)n_obs) ||
        !b.up(&dobs, obs, 3 * (size_t)n_obs) || !b.up(&dr, (const double*)nullptr, 3 * (size_t)n_obs) ||
        !b.up(&dj, (const double*)nullptr, 27 * (size_t)n_obs))
        return GBA_ERR_HIP;
    const long long lanes = 9LL * n_obs;
    hipLaunchKernelGGL(gba::vi::k_stereo_eval, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0,
                       nullptr, (long long)n_obs, ds, dpts, dkf, dpt, dobs, intr[0], intr[1], intr[2],
                       intr[3], intr[4], dr, dj);
    if (hipGetLastError() != hipSuccess) return GBA_ERR_HIP;
    if (hipMemcpy(r, dr, sizeof(double) * 3 * n_obs, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(J, dj, sizeof(double) * 27 * n_obs, hipMemcpyDeviceToHost) != hipSuccess)
        return GBA_ERR_HIP;
    return GBA_OK;
}

void gba_vi_default_options(gba_vi_options* o) {
    if (!o) return;
    o->pcg_max_iters = 100;
    o->solver = GBA_SOLVER_SCHUR;
    o->precision = GBA_FP64;
    o->reserved1 = 0;
    o->pcg_rejection_ratio = 0.0;
    o->pcg_tol = 1e-8;
    o->initial_lambda = 1e-4;
    o->min_diag = 1e-6;
    o->max_diag = 1e32;
}

gba_status gba_vi_solve(int device, const gba_vi_problem* prob, int max_iters, double tol,
                        const gba_vi_options* opts, gba_report* report, gba_trial* log, int max_log,
                        int* n_log) {
    using namespace gba::vi;
    const auto t_start = std::chrono::steady_clock::now();
    if (n_log) *n_log = 0;
    if (!prob || max_iters < 0 || !(tol >= 0.0) || (max_log > 0 && !log)) return GBA_ERR_INVALID_ARG;
    const gba_vi_problem& P = *prob;
    if (P.n_kf < 2 || P.n_pts < 0 || P.n_obs < 0 || !P.states || !P.intr || !P.pre ||
        (P.n_pts > 0 && !P.pts) || (P.n_obs > 0 && (!P.kf || !P.pt || !P.obs)) ||
        !(P.sigma_px > 0.0) || !(P.huber_delta2 >= 0.0) || !(P.sigma_gw > 0.0) || !(P.sigma_aw > 0.0))
        return GBA_ERR_INVALID_ARG;
    if (P.n_obs > INT32_MAX / 27 || P.n_pts > INT32_MAX || P.n_kf > INT32_MAX / 225)
        return GBA_ERR_UNSUPPORTED;
    gba_vi_options o;
    gba_vi_default_options(&o);
    if (opts) o = *opts;
    if (o.pcg_max_iters < 1 || !(o.pcg_tol >= 0.0) || !(o.initial_lambda > 0.0) ||
        (o.solver != GBA_SOLVER_SCHUR && o.solver != GBA_SOLVER_FULL) ||
        (o.precision != GBA_FP64 && o.precision != GBA_MIXED_FP32) ||

        !(o.min_diag > 0.0) || !(o.max_diag >= o.min_diag))
        return GBA_ERR_INVALID_ARG;
    if (P.n_pts == 0 && P.n_obs > 0) return GBA_ERR_UNKNOWN_ID;
    // Unknown ids are found on the device; where the call ends before that, they
    // are looked for here and name its status as they do otherwise.
    auto refuse = [&](gba_status st) {
        for (int64_t e = 0; e < P.n_obs; ++e)
            if (P.kf[e] < 0 || P.kf[e] >= P.n_kf || P.pt[e] < 0 || P.pt[e] >= P.n_pts) return (gba_status)GBA_ERR_UNKNOWN_ID;
        return st;
    };
    if (hipSetDevice(device) != hipSuccess) return refuse(GBA_ERR_HIP);
    const bool schur = o.solver == GBA_SOLVER_SCHUR;
    const int K = P.n_kf;
    const long long N = P.n_pts, M = P.n_obs, n = 15LL * K + 3 * N;
    const bool f32 = o.precision == GBA_MIXED_FP32;
    // one allocation for nearly everything: what is taken below in doubles a
    // keyframe and a point and bytes an observation (5 % pads), and for the
    // explicit blocks the pairs of a mean track and 20 blocks a keyframe
    const double track = N > 0 ? (double)M / (double)N : 0.0;
    const double per_obs = 76.0 + (schur ? (f32 ? 4.0 : 8.0) * 37 : 34.0);
    const double blocks = schur ? 300.0 * K * std::min(20.0, (double)K) + 8.0 * 0.65 * M * std::max(0.0, track - 1.0) : 0.0;
    gba::vi::DevBufs B((size_t)(8.0 * (1950.0 * K + 61.0 * N) + (double)M * per_obs + blocks + (1 << 20)));
    VIDev d{};
    d.K = K;
    d.N = N;
    d.M = M;
    auto grid = [](long long cnt) { return dim3((unsigned)std::max(1LL, (cnt + 255) / 256)); };
    const dim3 blk(256);
    hipError_t err = hipSuccess;
    auto chk = [&]() {
        if (err == hipSuccess) err = hipGetLastError();
        return err == hipSuccess;
    };
    const int* no_in = nullptr;
    // items (of in, or 0, 1, ...) sorted by key (0 .. nkeys - 1, stable; negative
    // keys left out), 12 bits a pass; tmp: as many items.  A workgroup places its items 64 at
    // a time in order, so short arrays are cut finer (109 us at 17,000 items
    // with 4096 each), as far as the counts stay within 4M.
    auto sort_by = [&](const int* in, int items, int kept, const int* key, int nkeys, int* out, int* tmp) {
        int passes = 1;
        while (((nkeys - 1) >> (kSortBits * passes)) > 0) ++passes;
        int *counts = nullptr, *total = nullptr;
        const int nb = std::min(nkeys, kSortBins);
        int per = 256;
        while (per < 4096 && (items / per + 1LL) * nb > (1 << 22)) per *= 2;
        const int nblk = (int)((items + (long long)per - 1) / per);
        if (!B.scratch(&counts, no_in, (size_t)nblk * nb) || !B.scratch(&total, no_in, (size_t)nb)) return false;
        int left = items;
        for (int p = 0; p < passes; ++p) {
            int* to = (passes - 1 - p) % 2 == 0 ? out : tmp;
            const int nbl = (int)((left + (long long)per - 1) / per), shift = kSortBits * p;
            hipLaunchKernelGGL(k_sort_count, dim3(nbl), blk, 0, nullptr, left, per, in, key, shift, nb, counts);
            hipLaunchKernelGGL(k_sort_rows, dim3(nb), dim3(64), 0, nullptr, nbl, counts, total);
            hipLaunchKernelGGL(k_sort_base, dim3(1), dim3(64), 0, nullptr, nb, total);
            hipLaunchKernelGGL(k_sort_place, dim3(nbl), dim3(64), 0, nullptr, left, per, in, key, shift, nb,
                               (const int*)counts, (const int*)total, to);
            in = to;
            left = kept;   // negative keys are gone after the first pass
        }
        return chk();
    };
    double *s15 = nullptr, *pre = nullptr, *x = nullptr, *r = nullptr, *z = nullptr, *pv = nullptr,
           *q = nullptr, *xb = nullptr, *p2 = nullptr, *Xraw = nullptr;
    int* pt_old = nullptr;
    std::vector<int> hlong, hlslot;
    long long Mp = 0, pairs = 0;   // padded point order; pairs of observations of one point
    bool twice = false;            // a keyframe observes a point more than once
    if (!B.up(&s15, P.states, 15 * (size_t)K) || !B.up(&pre, P.pre, (size_t)kPreStride * (K - 1)) ||
        !B.up(&Xraw, P.pts, 3 * (size_t)N) || !B.up(&d.X, (const double*)nullptr, 3 * (size_t)N) ||
        !B.up(&d.X_c, (const double*)nullptr, 3 * (size_t)N + 1) || !B.up(&pt_old, no_in, (size_t)N + 1))
        return refuse(GBA_ERR_OOM);
    {
        // The orders, on the device (gba_vi_order.h).  Points are renumbered
        // by the first keyframe that observes them (stable; unobserved points
        // last), so that a keyframe's observations and a run of consecutive
        // points touch nearby points and keyframes.
        const long long *kf64 = nullptr, *pt64 = nullptr;
        const double* raw = nullptr;
        int *kf = nullptr, *pt = nullptr, *first = nullptr, *cnt = nullptr, *cntn = nullptr, *renum = nullptr,
            *at = nullptr, *used = nullptr, *flag = nullptr, *tmp = nullptr;
        if (!B.scratch((long long**)&kf64, (const long long*)P.kf, (size_t)M) ||
            !B.scratch((long long**)&pt64, (const long long*)P.pt, (size_t)M) ||
            !B.scratch((double**)&raw, P.obs, 3 * (size_t)M) || !B.scratch(&kf, no_in, (size_t)M) || !B.scratch(&pt, no_in, (size_t)M) ||
            !B.scratch(&first, no_in, (size_t)N) || !B.scratch(&cnt, no_in, (size_t)N) || !B.scratch(&cntn, no_in, (size_t)N) ||
            !B.scratch(&renum, no_in, (size_t)N) || !B.scratch(&used, no_in, (size_t)N) || !B.scratch(&flag, no_in, 1) ||
            !B.scratch(&tmp, no_in, (size_t)std::max(N, M)))
            return refuse(GBA_ERR_OOM);
        std::vector<int> hcnt((size_t)N), hat((size_t)N + 1, 0);
        int h = 0;
        hipLaunchKernelGGL(k_vo_fill, dim3(1), blk, 0, nullptr, 1LL, flag, 0);
        if (N > 0) {
            hipLaunchKernelGGL(k_vo_fill, grid(N), blk, 0, nullptr, N, first, K);
            hipLaunchKernelGGL(k_vo_fill, grid(N), blk, 0, nullptr, N, cnt, 0);
            hipLaunchKernelGGL(k_vo_fill, grid(N), blk, 0, nullptr, N, used, 0);
            if (M > 0) hipLaunchKernelGGL(k_vo_raw, grid(M), blk, 0, nullptr, M, K, (int)N, kf64, pt64, kf, pt, first, cnt, flag);
            // ids that are not there end the call before they index anything
            if (!chk() || hipMemcpy(&h, flag, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return GBA_ERR_HIP;
            if (h != 0) return GBA_ERR_UNKNOWN_ID;
            if (!sort_by(no_in, (int)N, (int)N, first, K + 1, pt_old, tmp)) return GBA_ERR_HIP;
            hipLaunchKernelGGL(k_vo_points, grid(N), blk, 0, nullptr, (int)N, (const int*)pt_old, (const int*)cnt,
                               (const double*)Xraw, renum, cntn, d.X);
            if (!chk() || hipMemcpy(hcnt.data(), cntn, sizeof(int) * N, hipMemcpyDeviceToHost) != hipSuccess)
                return GBA_ERR_HIP;
        }
        // the padded point order: a point's observations sit in one wavefront
        // (64 slots) unless it has more than 64 of them
        for (long long j = 0; j < N; ++j) {
            const long long c = hcnt[(size_t)j];
            if (c > 64) hlong.push_back((int)j);
            else if (Mp % 64 + c > 64) Mp = (Mp + 63) / 64 * 64;
            hat[(size_t)j] = (int)Mp;
            pairs += c * (c - 1) / 2;
            Mp += c;
            if (Mp > INT32_MAX / 18) return GBA_ERR_UNSUPPORTED;
        }
        Mp = (Mp + 63) / 64 * 64;
        for (const int j : hlong)
            for (int c = 0; c < hcnt[(size_t)j]; ++c) hlslot.push_back(hat[(size_t)j] + c);
        int *qe = nullptr, *qs = nullptr, *qkf = nullptr, *qpt = nullptr, *key = nullptr, *dkf = nullptr, *dpt = nullptr,
            *ks = nullptr, *ko = nullptr;
        double *qobs = nullptr, *obs = nullptr;
        // (the kept ones first: they may open a chunk, and scratch stays behind)
        if (!B.up(&qkf, no_in, (size_t)Mp + 1) || !B.up(&qpt, no_in, (size_t)Mp + 1) ||
            !B.up(&key, no_in, (size_t)Mp) || !B.up(&qobs, (const double*)nullptr, 3 * (size_t)Mp + 1) ||
            !B.up(&dkf, no_in, (size_t)M + 1) || !B.up(&dpt, no_in, (size_t)M + 1) ||
            !B.up(&obs, (const double*)nullptr, 3 * (size_t)M + 1) || !B.up(&ks, no_in, (size_t)M) ||
            !B.up(&ko, no_in, (size_t)K + 1) || !B.scratch(&at, (const int*)hat.data(), (size_t)N) ||
            !B.scratch(&qe, no_in, (size_t)Mp) || !B.scratch(&qs, no_in, (size_t)Mp))
            return GBA_ERR_OOM;
        if (M > 0) {
            hipLaunchKernelGGL(k_vo_fill, grid(Mp + 1), blk, 0, nullptr, Mp + 1, qpt, -1);
            hipLaunchKernelGGL(k_vo_place, grid(M), blk, 0, nullptr, M, (const int*)pt, (const int*)renum,
                               (const int*)at, used, qe, qpt);
            hipLaunchKernelGGL(k_vo_rank, grid(Mp), blk, 0, nullptr, Mp, (const int*)qpt, (const int*)at,
                               (const int*)cntn, (const int*)kf, (const int*)qe, qs);
            if (!hlong.empty()) {
                const int nl = (int)hlslot.size();
                std::vector<int> hof((size_t)N, -1);
                for (size_t q = 0; q < hlong.size(); ++q) hof[(size_t)hlong[q]] = (int)q;
                int *of = nullptr, *key_kf = nullptr, *key_pt = nullptr, *by_kf = nullptr, *sorted = nullptr, *slot = nullptr;
                if (!B.scratch(&of, (const int*)hof.data(), (size_t)N) || !B.scratch(&key_kf, no_in, (size_t)M) ||
                    !B.scratch(&key_pt, no_in, (size_t)M) || !B.scratch(&by_kf, no_in, (size_t)nl) ||
                    !B.scratch(&sorted, no_in, (size_t)nl) || !B.scratch(&slot, (const int*)hlslot.data(), (size_t)nl))
                    return GBA_ERR_OOM;
                hipLaunchKernelGGL(k_vo_long_keys, grid(M), blk, 0, nullptr, M, (const int*)kf, (const int*)pt,
                                   (const int*)renum, (const int*)of, key_kf, key_pt);
                if (!sort_by(no_in, (int)M, nl, key_kf, K, by_kf, tmp) ||
                    !sort_by(by_kf, nl, nl, key_pt, (int)hlong.size(), sorted, tmp))
                    return GBA_ERR_HIP;
                hipLaunchKernelGGL(k_vo_long_place, grid(nl), blk, 0, nullptr, nl, (const int*)sorted, (const int*)slot, qs);
            }
            hipLaunchKernelGGL(k_vo_slots, grid(Mp), blk, 0, nullptr, Mp, (const int*)qs, (const int*)qpt,
                               (const int*)kf, raw, qkf, key, qobs, flag);
            if (!sort_by(no_in, (int)Mp, (int)M, key, K, ks, tmp)) return GBA_ERR_HIP;
            hipLaunchKernelGGL(k_vo_kf, grid(M), blk, 0, nullptr, (int)M, K, (const int*)ks, (const int*)qkf,
                               (const int*)qpt, (const double*)qobs, dkf, dpt, obs, key, ko);
            if (!chk() || hipMemcpy(&h, flag, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return GBA_ERR_HIP;
            twice = h != 0;
        }
        d.Mp = Mp;
        d.qkf = qkf;
        d.qpt = qpt;
        d.qobs = qobs;
        d.kf = dkf;
        d.pt = dpt;
        d.obs = obs;
        d.kslot = ks;
        d.kinv = key;
        d.kfoff = ko;
    }
    B.drop_scratch();
    if (!B.up(&d.st, (const double*)nullptr, kSt * (size_t)K) ||
        !B.up(&d.st_c, (const double*)nullptr, kSt * (size_t)K) ||
        !B.up(&d.info, (const double*)nullptr, 81 * (size_t)(K - 1)) ||
        !B.up(&d.ji, (const double*)nullptr, 216 * (size_t)(K - 1)) ||
        !B.up(&d.ri, (const double*)nullptr, 9 * (size_t)(K - 1)) ||
        !B.up(&d.b, (const double*)nullptr, (size_t)n) || !B.up(&d.hk, (const double*)nullptr, 225 * (size_t)K) ||
        !B.up(&d.hp, (const double*)nullptr, 9 * (size_t)N + 1) || !B.up(&d.dg, (const double*)nullptr, (size_t)n) ||
        !B.up(&d.mki, (const double*)nullptr, 225 * (size_t)K) || !B.up(&d.mp, (const double*)nullptr, 9 * (size_t)N + 1) ||
        !B.up(&d.scal, (const double*)nullptr, (size_t)kScalN) || !B.up(&x, (const double*)nullptr, (size_t)n) ||
        !B.up(&r, (const double*)nullptr, (size_t)n) || !B.up(&z, (const double*)nullptr, (size_t)n) ||
        !B.up(&pv, (const double*)nullptr, (size_t)n) || !B.up(&q, (const double*)nullptr, (size_t)n) ||
        !B.up(&xb, (const double*)nullptr, (size_t)n) || !B.up(&p2, (const double*)nullptr, schur ? 15 * (size_t)K : (size_t)n))
        return GBA_ERR_OOM;
    if (!schur) {
        d.w32 = f32 ? 1 : 0;
        if (!B.up(&d.jsp, (const double*)nullptr, 4 * (size_t)Mp + 1)) return GBA_ERR_OOM;
    }
    double* zb = nullptr;   // Schur form: the point vector of a product
    if (schur) {
        // W in FP32 takes half the doubles of FP64 (rounded up)
        d.w32 = o.precision == GBA_MIXED_FP32 ? 1 : 0;
        const size_t wn = (18 * 64 * (size_t)((M + 63) / 64) + 2) / (d.w32 ? 2 : 1);
        const size_t wpn = (18 * 64 * (size_t)(Mp / 64) + 2) / (d.w32 ? 2 : 1);
        int *lp = nullptr, *ls = nullptr;
        double *wk = nullptr, *wp = nullptr;
        if (!B.up(&wk, (const double*)nullptr, wn) || !B.up(&wp, (const double*)nullptr, wpn) ||
            !B.up(&d.icx, (const double*)nullptr, 135 * (size_t)(K - 1)) ||
            !B.up(&d.sm, (const double*)nullptr, 36 * (size_t)K) ||
            !B.up(&zb, (const double*)nullptr, 3 * (size_t)N + 1) ||
            !B.up(&lp, hlong.empty() ? (const int*)nullptr : hlong.data(), hlong.size()) ||
            !B.up(&ls, hlslot.empty() ? (const int*)nullptr : hlslot.data(), hlslot.size()) ||
            !B.up(&d.tb, (const double*)nullptr, 3 * (size_t)N + 1))
            return GBA_ERR_OOM;
        if (hipMemset(d.tb, 0, sizeof(double) * (3 * (size_t)N + 1)) != hipSuccess) return GBA_ERR_HIP;
        d.wk = wk;
        d.wp = wp;
        d.longp = lp;
        d.nlong = (int)hlong.size();
        d.lslot = ls;
        d.nlslot = (long long)hlslot.size();
    }
    // The visual blocks of S explicitly: when no keyframe observes a point
    // twice (the diagonal blocks are then exact), a keyframe's counts fit in
    // LDS, the pairs of observations can be listed, and vi_blocks_pay says so.
    bool explicit_s = schur && M > 0 && !twice && pairs > 0 && pairs <= 16 * M && K <= 16000;
    if (explicit_s) {
        (void)hipFuncSetAttribute((const void*)k_vi_s_pcg_one, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  144 * kOneKf * (kOneKf - 1));
        if (!B.up(&d.nrow, no_in, (size_t)K + 2) || !B.up(&d.nitem, no_in, (size_t)K + 1) ||
            !B.up(&d.items, (const int2*)nullptr, (size_t)pairs) || !B.up(&d.ad, (const double*)nullptr, 225 * (size_t)K) ||
            !B.up(&d.cb, (const double*)nullptr, 225 * (size_t)(K - 1)) ||
            !B.up(&d.cbt, (const double*)nullptr, 225 * (size_t)(K - 1)))
            explicit_s = false;   // no room for them: the implicit product needs none
    }
    if (explicit_s) {
        const int lds = K * (int)sizeof(int);
        hipLaunchKernelGGL(k_vi_pattern<false>, dim3(K), dim3(256), lds, nullptr, d);
        hipLaunchKernelGGL(k_vi_pattern_scan, dim3(1), dim3(1024), 0, nullptr, d);
        hipLaunchKernelGGL(k_vi_far, dim3((unsigned)((Mp + kFuseBlock - 1) / kFuseBlock)), dim3(kFuseBlock), 0, nullptr, d);
        int nf[2] = {0, 0};
        if (hipGetLastError() != hipSuccess ||
            hipMemcpy(nf, d.nrow + K, 2 * sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
            return GBA_ERR_HIP;
        d.nnz = nf[0];
        explicit_s = vi_blocks_pay(M, pairs, d.nnz, nf[1], o.pcg_max_iters);
    }
    if (explicit_s) {
        if (!B.up(&d.ncol, (const int*)nullptr, (size_t)d.nnz) || !B.up(&d.noff, (const int*)nullptr, (size_t)d.nnz) ||
            !B.up(&d.nkf, (const int*)nullptr, (size_t)d.nnz) ||
            !B.up(&d.vblk, (const double*)nullptr, 36 * (size_t)d.nnz))
            explicit_s = false;
    }
    if (explicit_s) {
        const int lds = K * (int)sizeof(int);
        hipLaunchKernelGGL(k_vi_pattern<true>, dim3(K), dim3(256), lds, nullptr, d);
        if (hipGetLastError() != hipSuccess) return GBA_ERR_HIP;
    }
    d.pre = pre;
    d.fx = P.intr[0];
    d.fy = P.intr[1];
    d.cx = P.intr[2];
    d.cy = P.intr[3];
    d.base = P.intr[4];
    d.inv_sigma = 1.0 / P.sigma_px;
    d.delta2 = P.huber_delta2;
    d.wg = 1.0 / (P.sigma_gw * P.sigma_gw);
    d.wa = 1.0 / (P.sigma_aw * P.sigma_aw);
    hipLaunchKernelGGL(k_vi_states_in, grid(K), blk, 0, nullptr, K, s15, d.st);
    hipLaunchKernelGGL(k_vi_info, grid(K - 1), blk, 0, nullptr, K - 1, pre, d.info);
    if (!chk()) return GBA_ERR_HIP;
    // the scalars: the PCG's, then the reduction slots' parts
    std::vector<double> hs((size_t)kScalN);
    auto read_scal = [&](long long cnt) {
        if (err == hipSuccess) err = hipMemcpy(hs.data(), d.scal, cnt * sizeof(double), hipMemcpyDeviceToHost);
        return err == hipSuccess;
    };
    // (each slot's parts summed in index order)
    auto red_sum = [&](int slot) {
        double t = 0.0;
        for (int i = 0; i < kPqParts; ++i) t += hs[(size_t)(kRedOff + slot * kPqParts + i)];
        return t;
    };
    auto red_parts = [&](int slot) { return d.scal + kRedOff + (long long)slot * kPqParts; };
    double* ps = d.scal + 8;   // PCG scalars
    // cost of (st, X) into its slot
    auto cost_of = [&](const double* st, const double* X) {
        hipLaunchKernelGGL(k_vi_cost, grid(M + K - 1), blk, 0, nullptr, d, st, X, (int)kRedCost);
    };
    auto linearize = [&]() {
        ZeroList zero;
        zero.add(d.b, n);
        zero.add(d.hk, 225LL * K);
        zero.add(d.hp, 9 * N + 1);
        hipLaunchKernelGGL(k_vi_clear, grid(zero.total()), blk, 0, nullptr, zero);
        if (M > 0) hipLaunchKernelGGL(k_vi_lin_stereo, grid(M), blk, 0, nullptr, d);
        if (M > 0) {
            if (d.w32) hipLaunchKernelGGL(k_vi_lin_stereo_pts<float>, grid(Mp), blk, 0, nullptr, d);
            else hipLaunchKernelGGL(k_vi_lin_stereo_pts<double>, grid(Mp), blk, 0, nullptr, d);
        }
        hipLaunchKernelGGL(k_vi_lin_inertial, grid(24LL * (K - 1)), blk, 0, nullptr, d);
        hipLaunchKernelGGL(k_vi_acc_inertial, grid(64LL * (K - 1)), blk, 0, nullptr, d);
        if (schur) hipLaunchKernelGGL(k_vi_cross, grid(225LL * (K - 1)), blk, 0, nullptr, d, explicit_s ? 1 : 0);
        return chk();
    };
    // z = sign C^-1 (B^T v + add) over the points (acc: -t . z added)
    auto schur_pts = [&](const double* v, const double* add, double sign, double* out, const double* g,
                         double* acc) {
        if (M == 0) return;
        double* none_q = nullptr;
        if (d.w32)
            hipLaunchKernelGGL((k_vi_schur_pts<float, false>), grid(Mp), blk, 0, nullptr, d, v, add, sign, out, g,
                               acc, none_q, 0.0);
        else
            hipLaunchKernelGGL((k_vi_schur_pts<double, false>), grid(Mp), blk, 0, nullptr, d, v, add, sign, out, g,
                               acc, none_q, 0.0);
        if (d.nlong > 0)
            hipLaunchKernelGGL(k_vi_long_pts, grid(d.nlong), blk, 0, nullptr, d, add, sign, out, g, acc);
    };
    // q = S v over the keyframes in one pass over the point-order W (the
    // point vector through zb): A v first, then the fused point pass adds
    // -B C^-1 B^T v; acc: v . S v
    // (out is zero on entry: cleared before the PCG and by each direction step)
    const dim3 fuse_grid((unsigned)((Mp + kFuseBlock - 1) / kFuseBlock + (15LL * K + kFuseBlock - 1) / kFuseBlock));
    auto schur_product = [&](const double* v, double* out, double lam, const double* g, double* acc) {
        const double* no_add = nullptr;
        if (d.w32)
            hipLaunchKernelGGL((k_vi_schur_pts<float, true>), fuse_grid, dim3(kFuseBlock), 0, nullptr, d, v, no_add,
                               1.0, zb, g, acc, out, lam);
        else
            hipLaunchKernelGGL((k_vi_schur_pts<double, true>), fuse_grid, dim3(kFuseBlock), 0, nullptr, d, v, no_add,
                               1.0, zb, g, acc, out, lam);
        if (d.nlong > 0) {
            hipLaunchKernelGGL(k_vi_long_pts, grid(d.nlong), blk, 0, nullptr, d, no_add, 1.0, zb, g, acc);
            if (d.w32) hipLaunchKernelGGL(k_vi_long_kf<float>, grid(d.nlslot), blk, 0, nullptr, d, (const double*)zb, out, g);
            else hipLaunchKernelGGL(k_vi_long_kf<double>, grid(d.nlslot), blk, 0, nullptr, d, (const double*)zb, out, g);
        }
    };
    // PCG from 0 to |r| <= pcg_tol |r0|: on (H + lam D) x = -b (full form),
    // or on S x_k = v followed by the point back-substitution (Schur form)
    const long long nn = schur ? 15LL * K : n;          // PCG unknowns
    // the PCG runs from its device scalars: its kernels are queued without
    // host round trips, and the stop flag is read every kPcgSync steps (a
    // read drains the queue); the first read comes kPcgSync steps before the
    // previous solve's count, as the next solve usually takes about as many
    constexpr int kPcgSync = 8;
    int prev_iters = 0;
    auto sync = [&](int it, bool& done) {
        const int first_read = std::max(kPcgSync, prev_iters - kPcgSync);
        if (it + 1 >= first_read && (it + 1 - first_read) % kPcgSync == 0 && it + 1 < o.pcg_max_iters) {
            if (!chk() || !read_scal(8 + kPcgScalars)) return false;
            done = hs[8 + kDone] != 0.0;
        }
        return true;
    };
    // Two launches a step take the host about 12 us, more than the kernels of a
    // short trajectory: after the first steps of a solve the Schur form replays
    // kGraphSteps steps as one graph.  The slots and the direction buffers of a
    // step repeat every six, so one recording from a multiple of six serves all.
    // (33 keyframes, 1,000 steps: 14.9 to 13.8 ms with the kernels' operands
    // requested ahead of their sums.)
    constexpr int kGraphSteps = 12, kGraphAfter = 24;
    static_assert(kGraphSteps % (2 * kSlots) == 0 && kGraphAfter % (2 * kSlots) == 0, "whole periods");
    StepGraph graph;
    const dim3 full_grid((unsigned)((Mp + kFuseBlock - 1) / kFuseBlock + (K + 6) / 8 + (n + kFuseBlock - 1) / kFuseBlock));
    const double ratio2 = (o.pcg_rejection_ratio > 0.0 && std::isfinite(o.pcg_rejection_ratio))
                              ? o.pcg_rejection_ratio * o.pcg_rejection_ratio : 0.0;
    auto pcg = [&](double lam) {
        const long long npt = schur ? 0 : N;   // points among the unknowns
        ZeroList zero;
        zero.add(x, n);
        zero.add(xb, nn);   // the best iterate: x0 = 0
        zero.add(d.scal, kScalN);
        zero.add(q, nn);   // the products add into q
        if (schur) {
            zero.add(d.sm, 36LL * K);
            zero.add(p2, nn);
        }
        hipLaunchKernelGGL(k_vi_begin, grid(N + nn + zero.total()), blk, 0, nullptr, d, lam, o.min_diag, o.max_diag,
                           nn, r, zb, zero);
        if (schur && M > 0) {   // r = -b_k + B C^-1 b_p
            if (d.w32) hipLaunchKernelGGL(k_vi_schur_blocks<float>, grid(M), blk, 0, nullptr, d, (const double*)zb, r);
            else hipLaunchKernelGGL(k_vi_schur_blocks<double>, grid(M), blk, 0, nullptr, d, (const double*)zb, r);
        }
        hipLaunchKernelGGL(k_vi_precond_kf, dim3((unsigned)((K + 3) / 4)), blk, 0, nullptr, d, lam, o.min_diag,
                           o.max_diag);
        hipLaunchKernelGGL(k_vi_apply_m, grid(15LL * K + npt), blk, 0, nullptr, d, npt, (const double*)r, z, pv,
                           ps + kAccN * (kSlots - 1));
        hipLaunchKernelGGL(k_vi_pcg_init, dim3(1), dim3(kPqParts), 0, nullptr, ps, o.pcg_tol, ratio2);
        if (explicit_s) {
            // the blocks of this step
            const dim3 fg((unsigned)d.nnz);
            if (d.nnz < 4096) {   // few blocks: four wavefronts each
                if (d.w32) hipLaunchKernelGGL((k_vi_form_blocks<float, 4>), fg, dim3(256), 0, nullptr, d);
                else hipLaunchKernelGGL((k_vi_form_blocks<double, 4>), fg, dim3(256), 0, nullptr, d);
            } else {
                if (d.w32) hipLaunchKernelGGL((k_vi_form_blocks<float, 1>), fg, dim3(64), 0, nullptr, d);
                else hipLaunchKernelGGL((k_vi_form_blocks<double, 1>), fg, dim3(64), 0, nullptr, d);
            }
        }
        if (explicit_s && K <= kOneKf) {
            hipLaunchKernelGGL(k_vi_s_pcg_one, dim3(1), dim3(kOneBlock), 144 * d.nnz, nullptr, d, ps, o.pcg_max_iters,
                               (const double*)r, (const double*)z, x);
        } else if (explicit_s || !schur) {
            // two launches per step: the product, with the decisions about
            // the step before, and the update
            const dim3 ug((unsigned)((K + 15) / 16 + (npt + kUpdPts - 1) / kUpdPts));
            double* dir[2] = {pv, p2};
            auto prod = [&](int it, bool last, hipStream_t on = nullptr) {
                const int slot = it % kSlots, prev = (it + kSlots - 1) % kSlots;
                if (schur)
                    hipLaunchKernelGGL(k_vi_s_prod, dim3((unsigned)((K + 3) / 4)), blk, 0, on, d, ps, slot, prev,
                                       it == 0 ? 1 : 0, last ? 1 : 0, (const double*)z,
                                       (const double*)dir[(it + 1) & 1], dir[it & 1], q, x, xb);
                else
                    hipLaunchKernelGGL(k_vi_full_prod, full_grid, dim3(kFuseBlock), 0, nullptr, d, lam, ps, slot, prev,
                                       last ? (int)kFullLast : it == 0 ? (int)kFullFirst : (int)kFullNext,
                                       (const double*)z, (const double*)dir[(it + 1) & 1], dir[it & 1], q, x, xb,
                                       (double*)nullptr);
            };
            auto step = [&](int it, hipStream_t on) {
                prod(it, false, on);
                hipLaunchKernelGGL(k_vi_s_update, ug, blk, 0, on, d, schur ? 0 : 1, ps, it % kSlots,
                                   (it + kSlots - 1) % kSlots, (const double*)dir[it & 1], q, x, r, z);
            };
            int it = 0;
            while (it < o.pcg_max_iters) {
                const bool whole = schur && it > 0 && it % (2 * kSlots) == 0 && it + kGraphSteps <= o.pcg_max_iters;
                if (whole && !graph.exec && !graph.failed && it >= kGraphAfter)
                    graph.record([&](hipStream_t on) {
                        for (int k = 0; k < kGraphSteps; ++k) step(2 * kSlots + k, on);
                    });
                bool done = false;
                if (whole && graph.exec) {
                    if (err == hipSuccess) err = hipGraphLaunch(graph.exec, nullptr);
                    it += kGraphSteps;
                    if (it >= prev_iters && it < o.pcg_max_iters) {   // (near or past the last solve's count)
                        if (!chk() || !read_scal(8 + kPcgScalars)) return false;
                        done = hs[8 + kDone] != 0.0;
                    }
                } else {
                    step(it, nullptr);
                    if (!sync(it, done)) return false;
                    it += 1;
                }
                if (done) break;
            }
            if (it == o.pcg_max_iters) prod(it, true);   // the decisions about the last step (or none: stopped)
        } else {
            const dim3 dirg((unsigned)std::max(1LL, std::min<long long>(1024, (nn + 255) / 256)));
            for (int it = 0; it < o.pcg_max_iters; ++it) {
                const int slot = it % kSlots;
                schur_product(pv, q, lam, ps, ps + kAccN * slot + kAccPq);   // p . q summed inside
                hipLaunchKernelGGL(k_vi_pcg_update, dim3((unsigned)((K + 15) / 16)), blk, 0, nullptr, d, ps, slot,
                                   (const double*)pv, (const double*)q, x, r, z);
                hipLaunchKernelGGL(k_vi_pcg_dir, dirg, blk, 0, nullptr, nn, ps, slot, (const double*)z, pv, x, xb, q);
                bool done = false;
                if (!sync(it, done)) return false;
                if (done) break;
            }
        }
        if (schur) {
            // x_p = -C^-1 (b_p + B^T x_k), and -(b_p + B^T x_k) . x_p
            schur_pts(x, d.b + 15 * (size_t)K, -1.0, x + 15 * (size_t)K, nullptr, red_parts(kRedCross));
        }
        return chk();
    };
    gba_report rep{};
    if (hipDeviceSynchronize() != hipSuccess) return GBA_ERR_HIP;
    rep.ms_other = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    rep.workspace_bytes = B.bytes;
    {
        ZeroList zero;
        zero.add(d.scal, kScalN);
        hipLaunchKernelGGL(k_vi_clear, grid(kScalN), blk, 0, nullptr, zero);
    }
    cost_of(d.st, d.X);
    if (!chk() || !read_scal(kScalN)) return GBA_ERR_HIP;
    double F = red_sum(kRedCost);
    rep.initial_cost = F;
    rep.termination = GBA_TERM_MAX_ITERS;
    int nl = 0;
    double lam = o.initial_lambda, nu = 2.0;
    if (!std::isfinite(F)) {
        rep.termination = GBA_TERM_NUMERICAL_FAILURE;
    } else if (max_iters > 0) {
        if (!linearize()) return GBA_ERR_HIP;
        for (int it = 0; it < max_iters; ++it) {
            if (!pcg(lam)) return GBA_ERR_HIP;
            // model decrease -(b.dx + 1/2 dx^T H dx) with the undamped H; in
            // the Schur form dx^T H dx = dx_k^T A dx_k + 2 dx_k^T B dx_p
            // + sum_j dx_j^T H_pp,j dx_j from the blocks, the middle term
            // from the back-substitution's (b_p + B^T dx_k) . dx_p; then the
            // candidate, its cost and |x|: one readback per trial
            if (!schur) {
                hipLaunchKernelGGL(k_vi_full_prod, full_grid, dim3(kFuseBlock), 0, nullptr, d, 0.0, ps, 0, 0,
                                   (int)kFullQuad, (const double*)x, (const double*)nullptr, (double*)nullptr,
                                   (double*)nullptr, (double*)nullptr, (double*)nullptr, red_parts(kRedQuad));
            }
            hipLaunchKernelGGL(k_vi_step, grid(16LL * K + N), blk, 0, nullptr, d, (const double*)x, schur ? 1 : 0);
            cost_of(d.st_c, d.X_c);
            if (!chk() || !read_scal(kScalN)) return GBA_ERR_HIP;
            const int iters = prev_iters = (int)hs[8 + kSteps];
            rep.pcg_iters_total += iters;
            const double cross = schur ? -red_sum(kRedCross) - red_sum(kRedBp) : 0.0;
            const double L = -(red_sum(kRedB) + 0.5 * (red_sum(kRedQuad) + 2.0 * cross));
            const double Fn = red_sum(kRedCost), xnorm = std::sqrt(red_sum(kRedX)), dnorm = std::sqrt(red_sum(kRedDx));
            const bool accepted = L > 0.0 && Fn < F;
            const double gain = L != 0.0 ? (F - Fn) / L : NAN;
            if (nl < max_log) log[nl++] = gba_trial{F, Fn, lam, L, dnorm, accepted ? 1 : 0, iters};
            rep.trials += 1;
            int stop = 0;
            if (accepted) {
                rep.accepted += 1;
                const double rel = (F - Fn) / F;
                std::swap(d.st, d.st_c);
                std::swap(d.X, d.X_c);
                F = Fn;
                lam *= std::max(1.0 / 3.0, 1.0 - std::pow(2.0 * gain - 1.0, 3));
                nu = 2.0;
                if (rel < tol) stop = GBA_TERM_COST_TOL;
            } else {
                lam *= nu;
                nu *= 2.0;
            }
            if (!stop && dnorm <= tol * (xnorm + tol)) stop = GBA_TERM_STEP_TOL;
            if (!stop && lam > 1e32) stop = GBA_TERM_LAMBDA_OVERFLOW;
            if (stop) {
                rep.termination = stop;
                break;
            }
            if (accepted && !linearize()) return GBA_ERR_HIP;
        }
    }
    rep.final_cost = F;
    rep.final_lambda = lam;
    hipLaunchKernelGGL(k_vi_states_out, grid(K), blk, 0, nullptr, K, d.st, s15);
    if (!chk()) return GBA_ERR_HIP;
    if (N > 0)
        hipLaunchKernelGGL(k_vo_points_out, grid(N), blk, 0, nullptr, (int)N, (const int*)pt_old, (const double*)d.X,
                           Xraw);
    if (!chk()) return GBA_ERR_HIP;
    if (hipMemcpy(P.states, s15, sizeof(double) * 15 * K, hipMemcpyDeviceToHost) != hipSuccess ||
        (N > 0 && hipMemcpy(P.pts, Xraw, sizeof(double) * 3 * N, hipMemcpyDeviceToHost) != hipSuccess))
        return GBA_ERR_HIP;
    rep.ms_total = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    if (report) *report = rep;
    if (n_log) *n_log = nl;
    return GBA_OK;
}

}  // extern "C"
