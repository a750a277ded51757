// Combined transition of a with-RF subsequence (Eq. 7) in FP64, with half the
// steps for pulses that are symmetric in time.
//
// U_j = D R_j, D = diag(E2, E2, E1); a step maps M to U_j M + (1 - E1) e_z M0.
// Let the waveform be symmetric (R_{N+1-j} = R_j) and its B1 have one phase, so
// that every B_j lies in one plane with e_z.  W, the rotation by pi about the
// transverse normal n of that plane, turns every B_j into -B_j and commutes with
// D, so U_j^T = R_j^T D = W D^{-1} U_j D W.  With P = U_M ... U_1 the product of the
// first half, the second half is
//   Q = U_1 ... U_M = W D P^T D^{-1} W,
// and its affine part sum_j U_1 ... U_{j-1} (1 - E1) e_z is
//   b_Q = -(1 - E1) / E1  W D s,   s = the sum over j < M of the z rows of
//                                      U_j ... U_1 (j = 0: e_z).
// So N / 2 steps, each with three more additions, replace N.
#pragma once

#include <hip/hip_runtime.h>

#include "consts.hpp"
#include "kernels.hpp"
#include "rotation.hpp"

namespace gbs {

// A stretch of steps: M -> a M + b M0, and the sum of the z rows of its partial
// products (before each of its steps).
struct Stretch {
    double a[3][4];  // [A | b]
    double s[3];
};

// What every step of one isochromat or group shares.
struct StepConst {
    double x, y, z, boff, e1, e2, e1m, gdt, k2;
};

// V = (D R) V0, then the T1 recovery toward M0
__device__ __forceinline__ void compose_step(const StepConst &c, const StepW &w, const double (&V0)[3][4],
                                             double (&V)[3][4]) {
    const double bx = w.b1r, by = w.b1i;
    const double bz = fma((double)w.gx, c.x, fma((double)w.gy, c.y, fma((double)w.gz, c.z, c.boff)));
    const double B2 = fma(bx, bx, fma(by, by, bz * bz));
    double ca, cb;  // R = (1 - cb |B|^2) I + ca [B]x + cb B B^T
    rot_coeffs(B2, c.gdt, c.k2, ca, cb);
    const double c0 = fma(-cb, B2, 1.0);
    const double qx = cb * bx, qy = cb * by, qz = cb * bz;
    const double pxy = qx * by, pxz = qx * bz, pyz = qy * bz;
    const double sx = ca * bx, sy = ca * by, sz = ca * bz;
    // rows of D R: transverse rows decay by E2, the z row by E1
    const double r00 = c.e2 * fma(qx, bx, c0), r01 = c.e2 * (pxy - sz), r02 = c.e2 * (pxz + sy);
    const double r10 = c.e2 * (pxy + sz), r11 = c.e2 * fma(qy, by, c0), r12 = c.e2 * (pyz - sx);
    const double r20 = c.e1 * (pxz - sy), r21 = c.e1 * (pyz + sx), r22 = c.e1 * fma(qz, bz, c0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double u0 = V0[0][k], u1 = V0[1][k], u2 = V0[2][k];
        V[0][k] = fma(r00, u0, fma(r01, u1, r02 * u2));
        V[1][k] = fma(r10, u0, fma(r11, u1, r12 * u2));
        V[2][k] = fma(r20, u0, fma(r21, u1, r22 * u2));
    }
    V[2][3] += c.e1m;
}

// Steps [lo, hi) of a waveform, two per iteration (T -> U -> T, so that the loop
// carries no register copies of the twelve entries).  SUMS: with the z rows.
template <bool SUMS>
__device__ __forceinline__ void compose_steps(const StepConst &c, const StepW *__restrict__ wave, int lo, int hi,
                                              Stretch &t) {
    double U[3][4];
    auto add = [&](const double (&V)[3][4]) {
        if (SUMS) {
#pragma unroll
            for (int k = 0; k < 3; ++k) t.s[k] += V[2][k];
        }
    };
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        t.s[r] = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) t.a[r][k] = r == k ? 1.0 : 0.0;
    }
    int j = lo;
    for (; j + 1 < hi; j += 2) {
        add(t.a);
        compose_step(c, wave[j], t.a, U);
        add(U);
        compose_step(c, wave[j + 1], U, t.a);
    }
    if (j < hi) {
        add(t.a);
        compose_step(c, wave[j], t.a, U);
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k) t.a[r][k] = U[r][k];
    }
}

// [A | b] of L after R
__device__ __forceinline__ void compose_after(const double (&L)[3][4], const double (&R)[3][4], double (&o)[3][4]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[r][k] = fma(L[r][0], R[0][k], fma(L[r][1], R[1][k], fma(L[r][2], R[2][k], k == 3 ? L[r][3] : 0.0)));
}

// The second half from the first (see above), n = (nx, ny, 0).
__device__ __forceinline__ void mirror(const StepConst &c, const Stretch &p, double nx, double ny, double (&q)[3][4]) {
    const double w00 = fma(2.0 * nx, nx, -1.0), w01 = 2.0 * nx * ny, w11 = fma(2.0 * ny, ny, -1.0);
    const double d[3] = {c.e2, c.e2, c.e1}, i[3] = {1.0 / c.e2, 1.0 / c.e2, 1.0 / c.e1};
    double g[3][3], h[3][3];  // D P^T D^{-1}
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) g[r][k] = d[r] * p.a[k][r] * i[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // W from the left
        h[0][k] = fma(w00, g[0][k], w01 * g[1][k]);
        h[1][k] = fma(w01, g[0][k], w11 * g[1][k]);
        h[2][k] = -g[2][k];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {  // and from the right
        q[r][0] = fma(h[r][0], w00, h[r][1] * w01);
        q[r][1] = fma(h[r][0], w01, h[r][1] * w11);
        q[r][2] = -h[r][2];
    }
    const double f = -c.e1m * i[2];
    const double s0 = c.e2 * p.s[0], s1 = c.e2 * p.s[1], s2 = c.e1 * p.s[2];
    q[0][3] = f * fma(w00, s0, w01 * s1);
    q[1][3] = f * fma(w01, s0, w11 * s1);
    q[2][3] = -f * s2;
}

// mirror divides by the decay of one step: sound while a step leaves a good part
// of M (any T1, T2 of more than a raster step).
__device__ __forceinline__ bool can_mirror(const StepConst &c) { return c.e1 > 0.25 && c.e2 > 0.25; }

// The whole transition of n_steps steps of a symmetric waveform from the
// stretch of its first n_steps / 2 (mid: its step n_steps / 2, for odd n_steps).
__device__ __forceinline__ void finish_mirrored(const StepConst &c, const StepW &mid, int n_steps, double nx,
                                                double ny, const Stretch &p, double (&o)[3][4]) {
    double q[3][4], m[3][4];
    mirror(c, p, nx, ny, q);
    if (n_steps & 1) {
        compose_step(c, mid, p.a, m);
        compose_after(q, m, o);
    } else {
        compose_after(q, p.a, o);
    }
}

}  // namespace gbs
