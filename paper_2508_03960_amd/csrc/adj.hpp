// Adjoint (reverse-mode) Bloch simulation: device-side layouts shared by
// k_adjoint.hip and api_adj.cpp.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace gbs {

constexpr int kAdjWG = 256;          // isochromats per workgroup (one per thread)
constexpr int kAdjSub = 8;           // ops per recomputed sub-segment (states in registers)
constexpr int kAdjMaxEvery = 256;    // largest checkpoint interval
constexpr int kAdjMaxClasses = 64;
constexpr int kAdjMaxRf = 3072;      // parameter-pulse samples (gradient accumulated in LDS, 24 KiB)

// One op of the flattened sequence: a raster step (Eq. A1, A2) or a
// relaxation block (Eq. 4, 5).  64 bytes.
struct AdjOp {
    float b1r, b1i, gx, gy, gz;  // raster: B1 [T] (unless param >= 0) and gradients [T/m]
    int32_t param;               // raster: sample of the parameter pulse, or -1
    int32_t kind;                // 0 raster step, 1 relaxation block
    int32_t pad;
    double tau;                  // relaxation: duration [s]
    double cyc[3];               // relaxation: gamma_bar * gradient moment [cycles/m]
};

struct AdjArgs {
    int64_t K;
    const float *x, *y, *z, *df, *m0;
    const int32_t *cls;
    const float *t1c, *t2c;
    int32_t n_classes;
    const AdjOp *ops;
    int32_t n_ops;
    const float2 *rfp;  // parameter pulse, n_rf samples
    int32_t n_rf;
    const int32_t *sstart;  // [n_ops + 2]: samples taken at boundary p are sid[sstart[p] .. sstart[p+1])
    const int32_t *sid;
    double dt;
    int32_t every;       // checkpoint interval in ops (multiple of kAdjSub, <= kAdjMaxEvery)
    float *ckpt;         // [n_ckpt][3][K]: state at boundaries 0, every, 2 every, ...
    float *sub;          // backward: [every / kAdjSub][3][K] sub-checkpoints of the current segment
    int32_t N;           // samples
    double2 *sig_part;   // forward: [grid][N] per-workgroup sums
    const double2 *w;    // backward: cotangent of the signal, [N] (d/dRe, d/dIm)
    float2 *grf_part;    // backward: [grid][n_rf]
    double2 *gt_part;    // backward: [grid][n_classes] (dL/dT1, dL/dT2)
};

// ---- by groups (k_adjgroup.hip) ---------------------------------------------
constexpr int kAdjSeg = 16;          // raster steps per segment of a pulse
constexpr int kAdjGroupMin = 4;      // isochromats per group from which the pulses are walked per group
constexpr int kAdjMinSteps = 128;    // raster steps (less one per pulse) from which they are

struct AdjStep {  // raster step of a pulse
    float b1r, b1i, gx, gy, gz;
    int32_t param;  // sample of the parameter pulse that replaces B1, or -1
};

struct AdjSeg {
    int32_t step0, n;  // steps [step0, step0 + n)
};

// One operation for the isochromats, and the samples at the boundary before it
// (list positions [sample0, sample0 + samples)); a closing entry holds the
// samples at the end.
struct AdjGOp {
    int32_t pulse;  // distinct pulse, or -1: relaxation
    int32_t coef;   // relaxations: their AdjGCoef
    int32_t sample0, samples;
};

struct AdjGCoef {  // a relaxation, once for all operations with the same numbers
    double tau, cyc[3];
};

struct AdjPulseArgs {
    int64_t G;
    const float4 *gtab;    // (x, y, z, dB0) of every group (coordinates that no pulse sees: 0)
    const int32_t *gcls;
    const float *t1c, *t2c;
    int32_t n_classes;
    const float2 *rfp;
    double dt;
    const AdjStep *steps;
    const AdjSeg *segs;    // [n_segs], pulse after pulse
    const int2 *pulses;    // [n_pulses] segments [x, y)
    int32_t n_pulses, n_segs;
    double *seg_t, *prefix, *suffix;  // [n_segs][12][G]
    double *total, *gsum;             // [n_pulses][12][G]
    double *tsum;                     // [n_segs][2][G]
    double *acc_rf, *acc_t;           // [n_rf][2], [n_classes][2]
};

struct AdjDecay {
    double e2, e1, om1;  // exp(-tau / T2), exp(-tau / T1), 1 - exp(-tau / T1)
};

struct AdjGroupArgs {
    int64_t K, G;
    const int32_t *order, *gid;  // [K] isochromats sorted by group, and their groups
    const float *x, *y, *z, *df, *m0;
    const int32_t *cls;
    const float *t1c, *t2c;
    int32_t n_classes;
    const AdjGOp *ops;  // [n_ops + 1]
    const AdjGCoef *coefs;
    int32_t n_ops;
    const int32_t *sid;
    int32_t every;
    float *ckpt, *sub;  // [n_ckpt][3][K], [every / kAdjSub][3][K]
    int32_t N;
    double2 *sig_part;  // [grid][N]
    const double2 *w;
    double2 *wl;        // [N] w in the order of the list
    double2 *gt_part;   // [grid][n_classes]
    const double *total;
    double *gsum;
    const AdjDecay *decay;  // [relaxations' coef][n_classes]
};

hipError_t launch_adjg_transitions(const AdjPulseArgs &a, hipStream_t st);
// fills decay
hipError_t launch_adjg_forward(const AdjGroupArgs &a, int n_coef, AdjDecay *decay, hipStream_t st);
hipError_t launch_adjg_backward(const AdjGroupArgs &a, const AdjPulseArgs &p, hipStream_t st);
hipError_t launch_adjg_results(const AdjPulseArgs &p, int n_rf, float *grad_rf, double *g1, double *g2, hipStream_t st);

// out[c] = sum over the rows r of part[r * n + c], in FP64
hipError_t launch_adj_rows(const double2 *part, int rows, int n, double *out, hipStream_t st);
hipError_t launch_adj_forward(const AdjArgs &a, hipStream_t st);
hipError_t launch_adj_backward(const AdjArgs &a, hipStream_t st);
hipError_t launch_adj_validate(int64_t K, const int32_t *cls, int n_classes, const float *t1c, const float *t2c,
                               int *flag, hipStream_t st);
hipError_t launch_adj_finalize(const AdjArgs &a, double *sig, float *grad_rf, double *grad_t1, double *grad_t2,
                               bool forward, hipStream_t st);
// g1, g2 <- sums of the rows [rows][C]
hipError_t launch_adj_class_rows(const double2 *part, int rows, int C, double *g1, double *g2, hipStream_t st);

}  // namespace gbs
