// The adjoint by groups, for phantoms where many isochromats share what a
// pulse sees (the coordinates along its gradients, T1, T2 and dB0).
//
// The sum over the isochromats of a group in a pulse's part of the gradient is
// bilinear in the state at its start, (M, M0), and the adjoint state lambda at
// its end: with P_j, Q_j the products of the pulse's steps before and after
// step j,
//   sum_iso v_j x mu_j = sum_k (R_j P_j e_k) x (D Q_j^T g_k),
//   g_k = sum_iso (M, M0)_k lambda,   k = 1 .. 4,
// so a group is as good as four isochromats that start from the unit vectors.
// The isochromats then take a pulse as one transition (k_adjg_forward,
// k_adjg_backward), the backward sweep adds up the 4 x 3 numbers g_k per
// group, over all blocks that play the same pulse, and the raster steps are
// walked once per distinct pulse and group, in FP64, in parallel over segments
// of kAdjSeg steps:
//  k_adjg_compose   the transition of every segment (FP64, three columns and
//                   the M0 column)
//  k_adjg_prefix    their products from the left: P at every segment's start,
//                   and the pulse's transition
//  k_adjg_suffix    the four g_k pulled back to every segment's end
//  k_adjg_gradient  back through every segment: dL/dB1 per step, and the T1, T2 terms
//  k_adjg_classes   those terms to the classes
// 1 M isochromats in 768 groups, 8 lines of a 3000-step pulse and 64 samples:
// forward 0.93 ms and backward 1.79 ms for the isochromats, 0.1 and 0.2 ms for the
// groups' steps, 0.4 ms for the grouping; stepped (k_adjoint.hip), 61 and 190 ms.
// Both isochromat kernels are bound by their chain of scalar loads and FP64 steps:
// operations of 16 bytes with their coefficients in a table that is read when
// they change, and cotangents in the list's order and an operation ahead, take
// 1.05 and 1.96 ms down to the figures above.
#include "adj.hpp"
#include "consts.hpp"
#include "device_math.hpp"

namespace gbs {

namespace {

typedef const __attribute__((address_space(4))) uint64_t *const_u64_ptr;

// element i of p in scalar registers (i uniform in the wavefront)
template <typename T>
__device__ __forceinline__ T uniform(const T *p, int64_t i) {
    static_assert(sizeof(T) % 8 == 0, "64-bit words");
    uint64_t w[sizeof(T) / 8];
    const const_u64_ptr q = (const_u64_ptr)(p + i);
#pragma unroll
    for (int j = 0; j < (int)(sizeof(T) / 8); ++j) w[j] = q[j];
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// S = sin t / t, C = (1 - cos t) / t^2, D = (t - sin t) / t^3 of t = sqrt(q):
// six terms of the series leave out less than 1e-17 below q = 1/16.
__device__ __forceinline__ void rot64(double q, double &S, double &C, double &D) {
    if (q <= 0.0625) {
        constexpr double f[14] = {1., 1., 1. / 2, 1. / 6, 1. / 24, 1. / 120, 1. / 720, 1. / 5040, 1. / 40320,
                                  1. / 362880, 1. / 3628800, 1. / 39916800, 1. / 479001600, 1. / 6227020800.};
        S = f[11];
        C = f[12];
        D = f[13];
#pragma unroll
        for (int k = 4; k >= 0; --k) {
            S = f[2 * k + 1] - q * S;
            C = f[2 * k + 2] - q * C;
            D = f[2 * k + 3] - q * D;
        }
    } else {
        const double t = sqrt(q);
        double sh, ch;
        sincos(0.5 * t, &sh, &ch);
        S = 2.0 * sh * ch / t;
        C = 2.0 * sh * sh / q;
        D = (1.0 - S) / q;
    }
}

struct Group {
    double x, y, z, kap, ofs, om1, om2;  // kap = 2 pi gamma_bar dt, ofs = 2 pi dB0 dt, om = 1 - exp(-dt / T)
};

__device__ __forceinline__ Group load_group(const AdjPulseArgs &a, int64_t g) {
    const float4 v = a.gtab[g];
    const int c = a.gcls[g];
    Group r;
    r.x = v.x;
    r.y = v.y;
    r.z = v.z;
    r.kap = kTwoPi * kGammaBar * a.dt;
    r.ofs = kTwoPi * (double)v.w * a.dt;
    r.om1 = -expm1(-a.dt / (double)a.t1c[c]);
    r.om2 = -expm1(-a.dt / (double)a.t2c[c]);
    return r;
}

struct Rot {
    double w[3], S, C, D;
    double R[3][3];
};

// The rotation of one raster step, w = -2 pi gamma_bar dt B and R = exp([w]x).
__device__ __forceinline__ Rot rotation(const AdjPulseArgs &a, const AdjStep &s, const Group &g) {
    double bx = s.b1r, by = s.b1i;
    if (s.param >= 0) {
        const float2 p = uniform(a.rfp, s.param);
        bx = p.x;
        by = p.y;
    }
    Rot r;
    r.w[0] = -g.kap * bx;
    r.w[1] = -g.kap * by;
    r.w[2] = -(g.kap * ((double)s.gx * g.x + (double)s.gy * g.y + (double)s.gz * g.z) + g.ofs);
    const double q = r.w[0] * r.w[0] + r.w[1] * r.w[1] + r.w[2] * r.w[2];
    rot64(q, r.S, r.C, r.D);
    const double c = 1.0 - r.C * q;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) r.R[i][k] = r.C * r.w[i] * r.w[k] + (i == k ? c : 0.0);
    r.R[0][1] -= r.S * r.w[2];
    r.R[1][0] += r.S * r.w[2];
    r.R[1][2] -= r.S * r.w[0];
    r.R[2][1] += r.S * r.w[0];
    r.R[2][0] -= r.S * r.w[1];
    r.R[0][2] += r.S * r.w[1];
    return r;
}

// R of a step applied to the four columns (relaxation follows).
__device__ __forceinline__ void rotate(const Rot &r, double (&P)[4][3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double x = P[k][0], y = P[k][1], z = P[k][2];
#pragma unroll
        for (int i = 0; i < 3; ++i) P[k][i] = r.R[i][0] * x + r.R[i][1] * y + r.R[i][2] * z;
    }
}
__device__ __forceinline__ void relax(const Group &g, double (&P)[4][3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        P[k][0] -= g.om2 * P[k][0];
        P[k][1] -= g.om2 * P[k][1];
        P[k][2] += g.om1 * ((k == 3 ? 1.0 : 0.0) - P[k][2]);
    }
}
__device__ __forceinline__ void load12(const double *p, int64_t G, double (&P)[4][3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i) P[k][i] = p[(3 * k + i) * G];
}
__device__ __forceinline__ void store12(double *p, int64_t G, const double (&P)[4][3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i) p[(3 * k + i) * G] = P[k][i];
}
__device__ __forceinline__ void unit12(double (&P)[4][3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i) P[k][i] = k == i ? 1.0 : 0.0;
}

}  // namespace

// Arrays of 12 doubles per (row, group): element 3 k + i of row r and group g at (12 r + 3 k + i) G + g.
__global__ __launch_bounds__(64) void k_adjg_compose(AdjPulseArgs a) {
    const int64_t g = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (g >= a.G) return;
    const AdjSeg s = uniform(a.segs, blockIdx.y);
    const Group grp = load_group(a, g);
    double P[4][3];
    unit12(P);
    for (int j = 0; j < s.n; ++j) {
        rotate(rotation(a, uniform(a.steps, s.step0 + j), grp), P);
        relax(grp, P);
    }
    store12(a.seg_t + 12 * (int64_t)blockIdx.y * a.G + g, a.G, P);
}

__global__ __launch_bounds__(64) void k_adjg_prefix(AdjPulseArgs a) {
    const int64_t g = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (g >= a.G) return;
    const int2 r = uniform(a.pulses, blockIdx.y);  // its segments
    double P[4][3], T[4][3], N[4][3];
    unit12(P);
    load12(a.seg_t + 12 * (int64_t)r.x * a.G + g, a.G, N);  // a segment ahead: the chain is a product, not a load
    for (int s = r.x; s < r.y; ++s) {
        __builtin_memcpy(T, N, sizeof(T));
        load12(a.seg_t + 12 * (int64_t)min(s + 1, r.y - 1) * a.G + g, a.G, N);
        store12(a.prefix + 12 * (int64_t)s * a.G + g, a.G, P);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = P[k][0], y = P[k][1], z = P[k][2];
#pragma unroll
            for (int i = 0; i < 3; ++i) P[k][i] = T[0][i] * x + T[1][i] * y + T[2][i] * z + (k == 3 ? T[3][i] : 0.0);
        }
    }
    store12(a.total + 12 * (int64_t)blockIdx.y * a.G + g, a.G, P);
}

__global__ __launch_bounds__(64) void k_adjg_suffix(AdjPulseArgs a) {
    const int64_t g = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (g >= a.G) return;
    const int2 r = uniform(a.pulses, blockIdx.y);
    double L[4][3], T[4][3], N[4][3];
    load12(a.gsum + 12 * (int64_t)blockIdx.y * a.G + g, a.G, L);
    load12(a.seg_t + 12 * (int64_t)(r.y - 1) * a.G + g, a.G, N);
    for (int s = r.y - 1; s >= r.x; --s) {
        __builtin_memcpy(T, N, sizeof(T));
        load12(a.seg_t + 12 * (int64_t)max(s - 1, r.x) * a.G + g, a.G, N);
        store12(a.suffix + 12 * (int64_t)s * a.G + g, a.G, L);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = L[k][0], y = L[k][1], z = L[k][2];
#pragma unroll
            for (int i = 0; i < 3; ++i) L[k][i] = T[i][0] * x + T[i][1] * y + T[i][2] * z;
        }
    }
}

// The states before each step of the segment are stepped again from its start
// for every step (kAdjSeg / 2 steps on average): the groups are few, and
// nothing is kept.
__global__ __launch_bounds__(64) void k_adjg_gradient(AdjPulseArgs a) {
    const int64_t g0 = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const bool act = g0 < a.G;
    const int64_t g = act ? g0 : a.G - 1;
    const AdjSeg s = uniform(a.segs, blockIdx.y);
    const Group grp = load_group(a, g);
    double L[4][3];
    load12(a.suffix + 12 * (int64_t)blockIdx.y * a.G + g, a.G, L);
    double t1 = 0.0, t2 = 0.0;
    for (int j = s.n - 1; j >= 0; --j) {
        double P[4][3];
        load12(a.prefix + 12 * (int64_t)blockIdx.y * a.G + g, a.G, P);
        for (int i = 0; i < j; ++i) {
            rotate(rotation(a, uniform(a.steps, s.step0 + i), grp), P);
            relax(grp, P);
        }
        const AdjStep st = uniform(a.steps, s.step0 + j);
        const Rot r = rotation(a, st, grp);
        rotate(r, P);  // v_k
        double c[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = P[k][0] - grp.om2 * P[k][0], y = P[k][1] - grp.om2 * P[k][1];
            const double m0 = k == 3 ? 1.0 : 0.0, dz = (P[k][2] - m0) - grp.om1 * (P[k][2] - m0);  // M'_z - M0
            t2 += L[k][0] * x + L[k][1] * y;
            t1 += L[k][2] * dz;
            const double mu[3] = {L[k][0] - grp.om2 * L[k][0], L[k][1] - grp.om2 * L[k][1], L[k][2] - grp.om1 * L[k][2]};
            c[0] += P[k][1] * mu[2] - P[k][2] * mu[1];
            c[1] += P[k][2] * mu[0] - P[k][0] * mu[2];
            c[2] += P[k][0] * mu[1] - P[k][1] * mu[0];
#pragma unroll
            for (int i = 0; i < 3; ++i) L[k][i] = r.R[0][i] * mu[0] + r.R[1][i] * mu[1] + r.R[2][i] * mu[2];
        }
        if (st.param >= 0) {  // wave-uniform
            const double ax = r.w[1] * c[2] - r.w[2] * c[1], ay = r.w[2] * c[0] - r.w[0] * c[2],
                         az = r.w[0] * c[1] - r.w[1] * c[0];
            const double bx = r.w[1] * az - r.w[2] * ay, by = r.w[2] * ax - r.w[0] * az;
            const double gx = act ? -grp.kap * (c[0] - r.C * ax + r.D * bx) : 0.0;
            const double gy = act ? -grp.kap * (c[1] - r.C * ay + r.D * by) : 0.0;
            const double sx = wave_sum_lane63_f64(gx), sy = wave_sum_lane63_f64(gy);
            if (threadIdx.x == 63) {
                atomicAdd(a.acc_rf + 2 * st.param, sx);
                atomicAdd(a.acc_rf + 2 * st.param + 1, sy);
            }
        }
    }
    if (act) {
        a.tsum[(2 * (int64_t)blockIdx.y) * a.G + g] = t1;
        a.tsum[(2 * (int64_t)blockIdx.y + 1) * a.G + g] = t2;
    }
}

__global__ __launch_bounds__(64) void k_adjg_classes(AdjPulseArgs a) {
    __shared__ double acc[kAdjMaxClasses][2];
    for (int i = threadIdx.x; i < 2 * kAdjMaxClasses; i += 64) acc[i >> 1][i & 1] = 0.0;
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (g < a.G) {
        double t1 = 0.0, t2 = 0.0;
#pragma unroll 8
        for (int s = 0; s < a.n_segs; ++s) {
            t1 += a.tsum[(2 * (int64_t)s) * a.G + g];
            t2 += a.tsum[(2 * (int64_t)s + 1) * a.G + g];
        }
        const int c = a.gcls[g];
        const double u1 = a.t1c[c], u2 = a.t2c[c];
        atomicAdd(&acc[c][0], t1 * a.dt / (u1 * u1));
        atomicAdd(&acc[c][1], t2 * a.dt / (u2 * u2));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * a.n_classes; i += 64)
        if (acc[i >> 1][i & 1] != 0.0) atomicAdd(a.acc_t + i, acc[i >> 1][i & 1]);
}

// ---- the isochromats -------------------------------------------------------
// One isochromat per thread, sorted by group; operations are relaxations (all
// raster steps without RF between two samples are one) and pulses.  State and
// adjoint state are FP64: a relaxation is 5 FP64 instructions, which issue at
// the rate of FP32 ones, where the stepped form's pairs (hi, lo) take 44.
// The coefficients of equal operations (the dwells of a readout) are computed
// once.  Both passes issue VALU instructions about half of the time, the rest
// are the operations' scalar work and the chains of five wavefronts per SIMD.
namespace {

struct IsoG {
    double x, y, z, df;
    float m0;
    int32_t cls, g;
};

__device__ __forceinline__ IsoG load_iso(const AdjGroupArgs &a, int64_t i, bool act) {
    IsoG s;
    const int32_t k = act ? a.order[i] : 0;
    s.x = a.x[k];
    s.y = a.y[k];
    s.z = a.z[k];
    s.df = a.df[k];
    s.m0 = act ? a.m0[k] : 0.f;
    s.cls = a.cls[k];
    s.g = act ? a.gid[i] : 0;
    return s;
}

struct RelaxG {
    double c, s, e1, r1;  // E2 cos, E2 sin of the phase of Eq. 4, E1, (1 - E1) M0
    double tau;
};

// (the decays, by duration and class, come from a table: their exponentials
// cost more than the rotation)
__device__ __forceinline__ RelaxG coefs_of(const AdjGroupArgs &a, const AdjGOp &op, const IsoG &s) {
    const AdjGCoef k = uniform(a.coefs, op.coef);
    const double cyc = k.cyc[0] * s.x + k.cyc[1] * s.y + k.cyc[2] * s.z + s.df * k.tau;
    const AdjDecay d = a.decay[(int64_t)op.coef * a.n_classes + s.cls];
    double sn, cs;
    sincospi(cyc - rint(cyc), &sn, &cs);  // half angle
    // 1 - cos and the decays' 1 - E in FP32, as the stepped form holds them: its
    // error is theirs (repeated by every dwell of a readout), and the two forms
    // agree on every phantom to the rounding of their sums
    const double c = 1.0 - (double)(float)(2.0 * sn * sn);
    return RelaxG{d.e2 * c, d.e2 * (2.0 * sn * cs), d.e1, d.om1 * s.m0, k.tau};
}

__device__ __forceinline__ void pulse_step(const AdjGroupArgs &a, int32_t id, const IsoG &s, double *M) {
    const double *T = a.total + 12 * (int64_t)id * a.G + s.g;
    double o[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        o[i] = T[i * a.G] * M[0] + T[(3 + i) * a.G] * M[1] + T[(6 + i) * a.G] * M[2] + T[(9 + i) * a.G] * (double)s.m0;
#pragma unroll
    for (int i = 0; i < 3; ++i) M[i] = o[i];
}

// Rotation by -phi about z (Eq. 4) and the decays.
__device__ __forceinline__ void relax_step(const RelaxG &r, double *M) {
    const double x = r.c * M[0] + r.s * M[1];
    M[1] = r.c * M[1] - r.s * M[0];
    M[0] = x;
    M[2] = r.e1 * M[2] + r.r1;
}

__device__ __forceinline__ void forward_op(const AdjGroupArgs &a, const AdjGOp &op, const IsoG &s, RelaxG &c,
                                           int32_t &have, double *M) {
    if (op.pulse >= 0) {
        pulse_step(a, op.pulse, s, M);
    } else {
        if (op.coef != have) {
            c = coefs_of(a, op, s);
            have = op.coef;
        }
        relax_step(c, M);
    }
}

}  // namespace

// the decays of every relaxation and class
__global__ void k_adjg_decay(const AdjGroupArgs a, int32_t n_coef, AdjDecay *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= (int64_t)n_coef * a.n_classes) return;
    const double t = a.coefs[i / a.n_classes].tau;
    const int c = (int)(i % a.n_classes);
    const double om1 = (float)-expm1(-t / (double)a.t1c[c]), om2 = (float)-expm1(-t / (double)a.t2c[c]);
    out[i] = AdjDecay{1.0 - om2, 1.0 - om1, om1};
}

// Samples (Eq. 6) wait in LDS, 8 of them for every lane of a wavefront; then a
// lane adds 16 lanes' part of one sample and component in FP64.  Against a DPP
// reduction per sample (24 instructions and two barriers each) 8 instructions a
// sample, and the sum over a wavefront's 64 isochromats is not rounded to FP32.
constexpr int kHeld = 8, kHeldPitch = 66;

__global__ __launch_bounds__(kAdjWG) __attribute__((amdgpu_waves_per_eu(5))) void k_adjg_forward(AdjGroupArgs a) {
    __shared__ float held[kAdjWG / 64][2][kHeld][kHeldPitch];
    __shared__ double2 sums[kAdjWG / 64][kHeld];
    const int64_t i = (int64_t)blockIdx.x * kAdjWG + threadIdx.x;
    const bool act = i < a.K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const IsoG s = load_iso(a, i, act);
    double M[3] = {0.0, 0.0, s.m0};
    RelaxG c{};
    int32_t have = -1;
    int first = 0, n_held = 0;  // samples [first, first + n_held) of the list wait
    auto flush = [&]() {        // uniform in the workgroup
        __syncthreads();
        const int n = lane & (kHeld - 1), comp = (lane >> 3) & 1, part = lane >> 4;
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) t += held[wave][comp][n][16 * part + j];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        const double im = __shfl_xor(t, 8);
        if (lane < kHeld) sums[wave][lane] = make_double2(t, im);
        __syncthreads();
        if ((int)threadIdx.x < n_held) {
            double re = 0.0, ie = 0.0;
#pragma unroll
            for (int w = 0; w < kAdjWG / 64; ++w) {
                re += sums[w][threadIdx.x].x;
                ie += sums[w][threadIdx.x].y;
            }
            a.sig_part[(int64_t)blockIdx.x * a.N + a.sid[first + threadIdx.x]] = make_double2(re, ie);
        }
        first += n_held;
        n_held = 0;
    };
    AdjGOp next = uniform(a.ops, 0);  // (a closing entry after the last)
    int left = 0;
    for (int p = 0;; ++p) {
        const AdjGOp op = next;
        if (p < a.n_ops) next = uniform(a.ops, p + 1);
        if (left == 0 && p < a.n_ops) {
            left = a.every;
            if (act) {
                float *q = a.ckpt + (int64_t)(p / a.every) * 3 * a.K + i;
                q[0] = (float)M[0];
                q[a.K] = (float)M[1];
                q[2 * a.K] = (float)M[2];
            }
        }
        --left;
        for (int n = 0; n < op.samples; ++n) {  // samples at this boundary
            held[wave][0][n_held][lane] = (float)M[0];
            held[wave][1][n_held][lane] = (float)M[1];
            if (++n_held == kHeld) flush();
        }
        if (p == a.n_ops) break;
        forward_op(a, op, s, c, have, M);
    }
    if (n_held) flush();
}

// The cotangents in the order in which the operations meet them.
__global__ void k_adjg_order(AdjGroupArgs a) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q < a.N) a.wl[q] = a.w[a.sid[q]];
}

// The samples at the boundary before op; first: the cotangent of the first one,
// loaded an operation ahead.
__device__ __forceinline__ void add_cotangent(const AdjGroupArgs &a, const AdjGOp &op, double2 first, double *L) {
    for (int n = 0; n < op.samples; ++n) {
        const double2 w = n ? uniform((const double2 *)a.wl, op.sample0 + n) : first;
        L[0] += w.x;
        L[1] += w.y;
    }
}
__device__ __forceinline__ double2 first_cotangent(const AdjGroupArgs &a, const AdjGOp &op) {
    return op.samples ? uniform((const double2 *)a.wl, op.sample0) : make_double2(0.0, 0.0);
}

// gsum[pulse][3 k + i][g] += sum over the wavefront's lanes of group g
__device__ __forceinline__ void add_group_sums(const AdjGroupArgs &a, int32_t pulse, const IsoG &s, bool act,
                                               const float *M, const double *L) {
    const double m[4] = {M[0], M[1], M[2], s.m0};
    uint64_t rest = __ballot(act);
    while (rest) {
        const int32_t g = __builtin_amdgcn_readlane(s.g, __builtin_ctzll(rest));
        const bool in = act && s.g == g;
        rest &= ~__ballot(in);
        double *out = a.gsum + 12 * (int64_t)pulse * a.G + g;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double t = wave_sum_lane63_f64(in ? m[k] * L[i] : 0.0);
                if ((threadIdx.x & 63) == 63) atomicAdd(out + (3 * k + i) * a.G, t);
            }
    }
}

// Back through every operation with lambda' behind it and lambda before it:
//   relaxations:  T2 += lambda'_xy . M'_xy tau,  T1 += lambda'_z (M'_z - M0) tau  (over T^2 at the end),
//                 lambda = the transpose of the operation's map, lambda';
//   pulses:       the group sums, and lambda = A^T lambda'.
__global__ __launch_bounds__(kAdjWG) __attribute__((amdgpu_waves_per_eu(5))) void k_adjg_backward(AdjGroupArgs a) {
    __shared__ double tg[kAdjMaxClasses][2];
    // of a sub-segment's operations: M'_x, M'_y, M'_z - M0 (relaxations) or the incoming state (pulses)
    __shared__ float V[kAdjSub][3][kAdjWG];
    const int tid = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * kAdjWG + tid;
    const bool act = i < a.K;
    for (int j = tid; j < kAdjMaxClasses * 2; j += kAdjWG) tg[j >> 1][j & 1] = 0.0;
    __syncthreads();
    const IsoG s = load_iso(a, i, act);
    double L[3] = {0.0, 0.0, 0.0};
    double x1 = 0.0, x2 = 0.0;
    RelaxG c{};
    int32_t have = -1;
    {
        const AdjGOp end = uniform(a.ops, a.n_ops);
        add_cotangent(a, end, first_cotangent(a, end), L);
    }
    const int n_seg = (a.n_ops + a.every - 1) / a.every;
    for (int seg = n_seg - 1; seg >= 0; --seg) {
        const int p0 = seg * a.every, p1 = min(p0 + a.every, a.n_ops);
        double M[3] = {0.0, 0.0, 0.0};
        auto load_state = [&](const float *q) {
            M[0] = q[0];
            M[1] = q[a.K];
            M[2] = q[2 * a.K];
        };
        if (act) load_state(a.ckpt + (int64_t)seg * 3 * a.K + i);
        const int last = p0 + (p1 - p0 - 1) / kAdjSub * kAdjSub;  // start of the last sub-segment
        if (a.every > kAdjSub) {  // step to the sub-segments' starts
            AdjGOp next = uniform(a.ops, p0);
            for (int p = p0; p <= last; ++p) {
                const AdjGOp op = next;
                next = uniform(a.ops, p + 1);
                if (act && ((p - p0) & (kAdjSub - 1)) == 0) {
                    float *q = a.sub + (int64_t)((p - p0) / kAdjSub) * 3 * a.K + i;
                    q[0] = (float)M[0];
                    q[a.K] = (float)M[1];
                    q[2 * a.K] = (float)M[2];
                }
                if (p < last) forward_op(a, op, s, c, have, M);
            }
        }
        for (int q0 = last; q0 >= p0; q0 -= kAdjSub) {
            const int q1 = min(q0 + kAdjSub, p1);
            if (act && a.every > kAdjSub) load_state(a.sub + (int64_t)((q0 - p0) / kAdjSub) * 3 * a.K + i);
            AdjGOp op = uniform(a.ops, q0);
            for (int p = q0; p < q1; ++p) {
                const AdjGOp next = uniform(a.ops, p + 1);
                float v[3] = {(float)M[0], (float)M[1], (float)M[2]};
                forward_op(a, op, s, c, have, M);
                if (op.pulse < 0) {
                    v[0] = (float)M[0];
                    v[1] = (float)M[1];
                    v[2] = (float)(M[2] - (double)s.m0);
                }
#pragma unroll
                for (int d = 0; d < 3; ++d) V[p - q0][d][tid] = v[d];
                op = next;
            }
            AdjGOp before = uniform(a.ops, q1 - 1);
            double2 wn = first_cotangent(a, before);
            for (int p = q1 - 1; p >= q0; --p) {
                op = before;
                const double2 w = wn;
                before = uniform(a.ops, max(p - 1, 0));
                wn = first_cotangent(a, before);
                float v[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) v[d] = V[p - q0][d][tid];
                if (op.pulse >= 0) {
                    add_group_sums(a, op.pulse, s, act, v, L);
                    const double *T = a.total + 12 * (int64_t)op.pulse * a.G + s.g;
                    const double x = L[0], y = L[1], z = L[2];
#pragma unroll
                    for (int d = 0; d < 3; ++d)
                        L[d] = T[3 * d * a.G] * x + T[(3 * d + 1) * a.G] * y + T[(3 * d + 2) * a.G] * z;
                } else {
                    if (op.coef != have) {
                        c = coefs_of(a, op, s);
                        have = op.coef;
                    }
                    x2 += (L[0] * v[0] + L[1] * v[1]) * c.tau;
                    x1 += L[2] * v[2] * c.tau;
                    const double x = c.c * L[0] - c.s * L[1];
                    L[1] = c.c * L[1] + c.s * L[0];
                    L[0] = x;
                    L[2] *= c.e1;
                }
                add_cotangent(a, op, w, L);
            }
        }
    }
    if (act) {
        const double t1 = a.t1c[s.cls], t2 = a.t2c[s.cls];
        atomicAdd(&tg[s.cls][0], x1 / (t1 * t1));
        atomicAdd(&tg[s.cls][1], x2 / (t2 * t2));
    }
    __syncthreads();
    for (int c2 = tid; c2 < a.n_classes; c2 += kAdjWG)
        a.gt_part[(int64_t)blockIdx.x * a.n_classes + c2] = make_double2(tg[c2][0], tg[c2][1]);
}

__global__ void k_adjg_results(int n_rf, int C, const double *__restrict__ acc_rf, const double *__restrict__ acc_t,
                               float *__restrict__ grad_rf, double *__restrict__ g1, double *__restrict__ g2) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < 2 * n_rf) grad_rf[j] = (float)acc_rf[j];
    if (j < C) {
        g1[j] += acc_t[2 * j];
        g2[j] += acc_t[2 * j + 1];
    }
}

hipError_t launch_adjg_transitions(const AdjPulseArgs &a, hipStream_t st) {
    if (a.n_pulses <= 0) return hipSuccess;
    const unsigned gb = (unsigned)((a.G + 63) / 64);
    hipLaunchKernelGGL(k_adjg_compose, dim3(gb, (unsigned)a.n_segs), dim3(64), 0, st, a);
    hipLaunchKernelGGL(k_adjg_prefix, dim3(gb, (unsigned)a.n_pulses), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_adjg_forward(const AdjGroupArgs &a, int n_coef, AdjDecay *decay, hipStream_t st) {
    const int64_t n = (int64_t)n_coef * a.n_classes;
    if (n > 0) hipLaunchKernelGGL(k_adjg_decay, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, a, n_coef, decay);
    hipLaunchKernelGGL(k_adjg_forward, dim3((unsigned)((a.K + kAdjWG - 1) / kAdjWG)), dim3(kAdjWG), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_adjg_backward(const AdjGroupArgs &a, const AdjPulseArgs &p, hipStream_t st) {
    if (a.N > 0) hipLaunchKernelGGL(k_adjg_order, dim3((unsigned)((a.N + 255) / 256)), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_adjg_backward, dim3((unsigned)((a.K + kAdjWG - 1) / kAdjWG)), dim3(kAdjWG), 0, st, a);
    if (p.n_pulses > 0) {
        const unsigned gb = (unsigned)((p.G + 63) / 64);
        hipLaunchKernelGGL(k_adjg_suffix, dim3(gb, (unsigned)p.n_pulses), dim3(64), 0, st, p);
        hipLaunchKernelGGL(k_adjg_gradient, dim3(gb, (unsigned)p.n_segs), dim3(64), 0, st, p);
        hipLaunchKernelGGL(k_adjg_classes, dim3(gb), dim3(64), 0, st, p);
    }
    return hipGetLastError();
}

hipError_t launch_adjg_results(const AdjPulseArgs &p, int n_rf, float *grad_rf, double *g1, double *g2, hipStream_t st) {
    const int n = 2 * n_rf > p.n_classes ? 2 * n_rf : p.n_classes;
    hipLaunchKernelGGL(k_adjg_results, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n_rf, p.n_classes, p.acc_rf,
                       p.acc_t, grad_rf, g1, g2);
    return hipGetLastError();
}

}  // namespace gbs
