// Two-axis (x, z) groups on gfx950: the runs of the group-sorted layout and
// one combined transition per run for Gx+Gz with-RF subsequences.
//
// k_compose_pair: 64 runs per workgroup, one per lane; each wavefront composes a
// segment of the steps in FP64 (the same step as the per-isochromat composition
// of the cached method, with the run's x, z, T1, T2, dB0; the waveform values
// are wave-uniform scalar loads), and the first one multiplies the segments.
// The steps are a serial chain of FP64 latencies: with one wavefront per 64 runs
// 57,000 runs leave one wavefront per SIMD (1.00 ms for 3000 steps); segments
// give each SIMD several.  Symmetric pulses take half the steps (compose.hpp).
#include "compose.hpp"
#include "consts.hpp"
#include "pairs.hpp"
#include "rotation.hpp"

namespace gbs {

__global__ void k_run_table(int64_t n_runs, const int32_t *__restrict__ first, const float *__restrict__ xi,
                            const float *__restrict__ zi, const float *__restrict__ t1i,
                            const float *__restrict__ t2i, const float *__restrict__ dfi, float4 *__restrict__ rtab,
                            float *__restrict__ rz) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n_runs;
         r += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = 4 * (int64_t)first[r];  // a run starts with a real isochromat
        rtab[r] = make_float4(xi[k], t1i[k], t2i[k], dfi[k]);
        rz[r] = zi[k];
    }
}

__device__ __forceinline__ void pair_segment(const StepConst &c, const StepW *wave, int n, bool half, int seg, int S,
                                            Stretch &t) {
    const int m = half ? n / 2 : n;
    const int lo = (int)((int64_t)m * seg / S), hi = (int)((int64_t)m * (seg + 1) / S);
    if (half)
        compose_steps<true>(c, wave, lo, hi, t);
    else
        compose_steps<false>(c, wave, lo, hi, t);
}

__global__ __launch_bounds__(512) void k_compose_pair(int64_t n_runs, const float4 *__restrict__ rtab,
                                                       const float *__restrict__ rz, const StepW *__restrict__ wave,
                                                       int32_t n_steps, double dt, WaveSym sym, double *__restrict__ out) {
    extern __shared__ double seg_sum[];  // [segment - 1][15][lane]
    const int seg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, S = blockDim.x >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * 64 + lane, r = r0 < n_runs ? r0 : n_runs - 1;
    const float4 g = rtab[r];
    const double t1 = g.y, t2 = g.z;
    const double gdt = kTwoPi * kGammaBar * dt;
    const StepConst c{g.x, 0.0, rz[r], (double)g.w / kGammaBar, exp(-dt / t1), exp(-dt / t2), -expm1(-dt / t1), gdt,
                      gdt * gdt};
    const bool half = sym.sym && __all(can_mirror(c));  // (the same in all wavefronts: they hold the same runs)
    Stretch t;
    pair_segment(c, wave, n_steps, half, seg, S, t);
    if (S > 1) {
        double *mine = seg_sum + (int64_t)(seg - 1) * 15 * 64 + lane;
        if (seg > 0) {
#pragma unroll
            for (int i = 0; i < 12; ++i) mine[64 * i] = t.a[i / 4][i % 4];
#pragma unroll
            for (int i = 0; i < 3; ++i) mine[64 * (12 + i)] = t.s[i];
        }
        __syncthreads();
        if (seg > 0) return;
        for (int q = 1; q < S; ++q) {  // the later segment on the left
            const double *o = seg_sum + (int64_t)(q - 1) * 15 * 64 + lane;
            double L[3][4], R[3][4];
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                L[i / 4][i % 4] = o[64 * i];
                R[i / 4][i % 4] = t.a[i / 4][i % 4];
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)
                t.s[k] += o[64 * 12] * R[0][k] + o[64 * 13] * R[1][k] + o[64 * 14] * R[2][k];
            compose_after(L, R, t.a);
        }
    }
    if (r0 >= n_runs) return;
    double T[3][4];
    if (half) {
        finish_mirrored(c, wave[n_steps / 2], n_steps, sym.nx, sym.ny, t, T);
    } else {
#pragma unroll
        for (int i = 0; i < 12; ++i) T[i / 4][i % 4] = t.a[i / 4][i % 4];
    }
    double *o = out + 12 * r;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int k = 0; k < 3; ++k) o[3 * i + k] = T[i][k];
        o[9 + i] = T[i][3];
    }
}

static dim3 grid_of(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return dim3((unsigned)g);
}

hipError_t launch_run_table(int64_t n_runs, const int32_t *first, const float *xi, const float *zi,
                            const float *t1i, const float *t2i, const float *dfi, float4 *rtab, float *rz,
                            hipStream_t st) {
    if (n_runs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_run_table, grid_of(n_runs), dim3(256), 0, st, n_runs, first, xi, zi, t1i, t2i, dfi, rtab, rz);
    return hipGetLastError();
}

hipError_t launch_compose_pair(int64_t n_runs, const float4 *rtab, const float *rz, const StepW *wave,
                               int32_t n_steps, double dt, const WaveSym &sym, double *out, hipStream_t st) {
    if (n_runs <= 0) return hipSuccess;
    const int64_t blocks = (n_runs + 63) / 64;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    int S = 1;  // segments: up to 8, until there are four wavefronts per SIMD, each with at least 32 steps
    while (S < 8 && blocks * S < 4096 && n_steps / (4 * S) >= 32) S *= 2;
    const size_t lds = sizeof(double) * 15 * 64 * (size_t)(S - 1);
    hipLaunchKernelGGL(k_compose_pair, dim3((unsigned)blocks), dim3(64 * S), lds, st, n_runs, rtab, rz, wave, n_steps, dt,
                       sym, out);
    return hipGetLastError();
}

}  // namespace gbs
