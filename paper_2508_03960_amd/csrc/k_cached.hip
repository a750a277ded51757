// The conventional accelerated method on gfx950 (Sec. 2.2), the comparator
// of the grouped update.
//
// k_cached: one thread per isochromat.  In compose mode the thread multiplies
// its 3x4 homogeneous transition [A | b] (M' = A M + b M0) by D R for every
// raster step of the block in FP64 (Eq. 7 with U = D R of Eq. A1, A2; the
// step's waveform values are wave-uniform scalar loads), rounds it to FP32
// into the cache and applies it (half the steps for symmetric pulses,
// compose.hpp).  Later occurrences of the same waveform read
// the 48 cached bytes instead (dynamic caching).  The state between operations
// is FP64, 24 bytes per isochromat.
//
// k_direct_adc: Eq. (6) with Eq. (4), (5) evaluated for every (isochromat,
// sample) pair of a with-ADC block without RF.  Thread t of a workgroup owns
// sample t mod ns, and the slice t / ns of the isochromats when ns < 256.
// Isochromats pass through LDS in chunks of 256 and are read as broadcasts,
// so every thread keeps its sample's sum in registers and no cross-lane
// reduction runs per sample.  The phase is formed and reduced modulo one cycle
// in FP64 and evaluated with the hardware sin/cos; the T2 decay uses the
// hardware exp2.
//
// k_adc_product: the same for samples arithmetic in n, as a matrix product.
#include <algorithm>

#include "cached.hpp"
#include "compose.hpp"
#include "consts.hpp"
#include "device_math.hpp"
#include "rotation.hpp"

namespace gbs {

constexpr int kCachedBlock = 256;
constexpr int kAdcBlock = 256;
constexpr int kAdcMaxGrid = 2048;  // 8 workgroups per CU on 256 CUs
constexpr double kLog2e = 1.44269504088896340736;

template <int MODE>
__global__ __launch_bounds__(kCachedBlock) void k_cached(CachedArgs a) {
    const int64_t k = (int64_t)blockIdx.x * kCachedBlock + threadIdx.x;
    if (k >= a.K) return;
    if (a.gate && *a.gate != a.gate_value) return;
    const int64_t K = a.K;
    const double m0 = a.ph.m0[k];
    double vx, vy, vz;
    if (a.s64_in) {
        vx = a.s64_in[k];
        vy = a.s64_in[K + k];
        vz = a.s64_in[2 * K + k];
    } else if (a.min_x) {
        vx = a.min_x[k];
        vy = a.min_y[k];
        vz = a.min_z[k];
    } else {
        vx = 0.0;
        vy = 0.0;
        vz = m0;
    }
    if (a.has_pre) {  // Eq. (4), (5); phase reduced modulo one cycle in FP64
        const double x = a.ph.x[k], y = a.ph.y[k], z = a.ph.z[k], df = a.ph.df[k];
        const double cyc = fma(a.pre_cyc[0], x, fma(a.pre_cyc[1], y, fma(a.pre_cyc[2], z, df * a.pre_tau)));
        double sn, cs;
        sincos(kTwoPi * (cyc - rint(cyc)), &sn, &cs);
        const double e2 = exp(-a.pre_tau / (double)a.ph.t2[k]);
        const double e1 = exp(-a.pre_tau / (double)a.ph.t1[k]);
        const double nx = e2 * (vx * cs + vy * sn);
        const double ny = e2 * (vy * cs - vx * sn);
        vx = nx;
        vy = ny;
        vz = m0 + (vz - m0) * e1;
    }
    if (MODE == kCacheApply) {
        const float4 r0 = a.cache[k], r1 = a.cache[K + k], r2 = a.cache[2 * K + k];
        const double nx = fma((double)r0.x, vx, fma((double)r0.y, vy, fma((double)r0.z, vz, (double)r0.w * m0)));
        const double ny = fma((double)r1.x, vx, fma((double)r1.y, vy, fma((double)r1.z, vz, (double)r1.w * m0)));
        const double nz = fma((double)r2.x, vx, fma((double)r2.y, vy, fma((double)r2.z, vz, (double)r2.w * m0)));
        vx = nx;
        vy = ny;
        vz = nz;
    } else if (MODE == kCacheCompose) {
        const double t1 = a.ph.t1[k], t2 = a.ph.t2[k];
        // (off-resonance as a field, T)
        const StepConst c{a.ph.x[k], a.ph.y[k], a.ph.z[k], (double)a.ph.df[k] / kGammaBar, exp(-a.dt / t1), exp(-a.dt / t2),
                          -expm1(-a.dt / t1), a.gdt, a.gdt * a.gdt};
        Stretch st;
        double T[3][4];
        if (a.sym.sym && __all(can_mirror(c))) {
            compose_steps<true>(c, a.wave, 0, a.n_steps / 2, st);
            finish_mirrored(c, a.wave[a.n_steps / 2], a.n_steps, a.sym.nx, a.sym.ny, st, T);
        } else {
            compose_steps<false>(c, a.wave, 0, a.n_steps, st);
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) T[r][q] = st.a[r][q];
        }
        a.cache[k] = make_float4((float)T[0][0], (float)T[0][1], (float)T[0][2], (float)T[0][3]);
        a.cache[K + k] = make_float4((float)T[1][0], (float)T[1][1], (float)T[1][2], (float)T[1][3]);
        a.cache[2 * K + k] = make_float4((float)T[2][0], (float)T[2][1], (float)T[2][2], (float)T[2][3]);
        const double nx = fma(T[0][0], vx, fma(T[0][1], vy, fma(T[0][2], vz, T[0][3] * m0)));
        const double ny = fma(T[1][0], vx, fma(T[1][1], vy, fma(T[1][2], vz, T[1][3] * m0)));
        const double nz = fma(T[2][0], vx, fma(T[2][1], vy, fma(T[2][2], vz, T[2][3] * m0)));
        vx = nx;
        vy = ny;
        vz = nz;
    }
    if (a.s64_out) {
        a.s64_out[k] = vx;
        a.s64_out[K + k] = vy;
        a.s64_out[2 * K + k] = vz;
    } else {
        a.mout_x[k] = (float)vx;
        a.mout_y[k] = (float)vy;
        a.mout_z[k] = (float)vz;
    }
}

template <bool COILS>
__global__ __launch_bounds__(kAdcBlock) void k_direct_adc(DirectAdcArgs a) {
    constexpr int MC = COILS ? kMaxCoils : 1;
    __shared__ double4 pos[kAdcBlock];  // x, y, z, df
    __shared__ float4 mag[kAdcBlock];   // Mx, My, -log2(e) / T2, 0
    __shared__ float2 sen[MC][kAdcBlock];  // S(k, p) of the chunk (coils only)
    __shared__ double2 red[kAdcBlock];
    const int t = threadIdx.x;
    const int ns = a.n_samples;
    const int P = COILS ? a.n_coils : 1;
    const int G = kAdcBlock / ns;  // isochromat slices per chunk
    const int cnt = kAdcBlock / G;
    const int n = t % ns, g = t / ns;
    const bool active = g < G;
    const double4 c = active ? a.samp[n] : make_double4(0.0, 0.0, 0.0, 0.0);
    const float tau = (float)c.w;
    const int64_t K = a.K;
    double acc_re[MC], acc_im[MC];
#pragma unroll
    for (int p = 0; p < MC; ++p) acc_re[p] = acc_im[p] = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kAdcBlock; base < K; base += (int64_t)gridDim.x * kAdcBlock) {
        const int64_t k = base + t;
        double4 q0 = make_double4(0.0, 0.0, 0.0, 0.0);
        float4 m = make_float4(0.f, 0.f, 0.f, 0.f);  // padding slots add nothing
        if (k < K) {
            q0 = make_double4(a.ph.x[k], a.ph.y[k], a.ph.z[k], a.ph.df[k]);
            float mx = 0.f, my = 0.f;
            if (a.s64_in) {
                mx = (float)a.s64_in[k];
                my = (float)a.s64_in[K + k];
            } else if (a.min_x) {
                mx = a.min_x[k];
                my = a.min_y[k];
            }
            m = make_float4(mx, my, (float)(-kLog2e / (double)a.ph.t2[k]), 0.f);
        }
        __syncthreads();  // the previous chunk has been read
        pos[t] = q0;
        mag[t] = m;
        if (COILS) {
#pragma unroll
            for (int p = 0; p < MC; ++p)
                if (p < P) sen[p][t] = k < K ? make_float2(a.coil_re[p * K + k], a.coil_im[p * K + k])
                                             : make_float2(0.f, 0.f);
        }
        __syncthreads();
        if (active) {
            float sr[MC], si[MC];
#pragma unroll
            for (int p = 0; p < MC; ++p) sr[p] = si[p] = 0.f;
            auto add = [&](int j) {
                const double4 q = pos[j];
                const float4 v = mag[j];
                const double cyc = fma(c.x, q.x, fma(c.y, q.y, fma(c.z, q.z, c.w * q.w)));
                float s, co;
                sincos_rev(cyc, &s, &co);
                const float e = __builtin_amdgcn_exp2f(tau * v.z);  // exp(-tau / T2)
                // (Mx + i My) exp(-i 2 pi cyc)
                const float tr = e * fmaf(v.x, co, v.y * s), ti = e * fmaf(v.y, co, -v.x * s);
                if (COILS) {
#pragma unroll
                    for (int p = 0; p < MC; ++p)
                        if (p < P) {
                            const float2 w = sen[p][j];
                            sr[p] = fmaf(tr, w.x, fmaf(-ti, w.y, sr[p]));
                            si[p] = fmaf(tr, w.y, fmaf(ti, w.x, si[p]));
                        }
                } else {
                    sr[0] += tr;
                    si[0] += ti;
                }
            };
            // slice g takes chunk entries g, g + G, ...: cnt of them (a
            // wave-uniform count), and one more when 256 is not a multiple of G
#pragma unroll 4
            for (int i = 0; i < cnt; ++i) add(g + i * G);
            if (g + cnt * G < kAdcBlock) add(g + cnt * G);
#pragma unroll
            for (int p = 0; p < MC; ++p) {
                acc_re[p] += sr[p];
                acc_im[p] += si[p];
            }
        }
    }
#pragma unroll
    for (int p = 0; p < MC; ++p) {
        if (p >= P) break;
        if (p > 0) __syncthreads();  // the previous coil's sums have been read
        red[t] = make_double2(acc_re[p], acc_im[p]);
        __syncthreads();
        if (t < ns) {
            double re = 0.0, im = 0.0;
            for (int q = 0; q < G; ++q) {
                re += red[q * ns + t].x;
                im += red[q * ns + t].y;
            }
            a.partial[((int64_t)p * gridDim.x + blockIdx.x) * ns + t] = make_double2(re, im);
        }
    }
}

// ---------------------------------------------------------------- k_adc_product
// Sample n = i + 16 j of isochromat k is A_i B_j with A_i = z^i, B_j = M f z^{16 j}
// (z: phase and decay of one sample step, f: of the first sample), so up to 256
// samples are a complex 16 x 16 product over the isochromats: two row tiles
// {Re, Im} A_{0..7}, A_{8..15} and two column tiles {Re, Im} B_{0..7}, B_{8..15},
// four v_mfma_f32_16x16x4_f32 per four isochromats (samples <= 128: two).  A
// wavefront takes 32 isochromats at a time: lane l makes the 16 values of A
// (l < 32) or B of isochromat l % 32, each directly (phase reduced in FP64,
// hardware sin/cos and exp2, as k_direct_adc per sample), and leaves them in
// LDS for the lanes of the product.  Per isochromat that is 32 evaluations in
// place of 256; the rest is 32 cycles of the matrix core per SIMD.  The 32
// isochromats of a chunk add in the matrix core, FP64 from there.
// A term here holds up to two sine/cosine pairs, each short by kTurnBias on
// average, where k_direct_adc's holds one, and a sum over many isochromats shows
// it: M makes up for both.  Phases of 0 are exact: an isochromat whose phase
// stands still gets nothing, and the sums with A_0 = 1 give one pair's share back.
// Errors of the signal, k_direct_adc and this: 66 k isochromats of a brain phantom,
// 48 samples 5.1e-8 and 3.5e-8 (9.0e-8 with neither blocks nor this), 256 samples
// 9.0e-8 and 5.0e-8; 2.07 M, FSE of 8 x 16 lines of 256, eight seeds: 9.9e-8 and
// 7.5e-8.  2.1M isochromats: 67 us for 48 to 128 samples (65 with 256 isochromats
// between FP64 sums), 85 for 256 (83).
typedef float cached_f32x4 __attribute__((ext_vector_type(4)));
constexpr int kProdChunk = 32;
constexpr int kProdPad = 36;                  // floats per isochromat and side; 32 used (36: 16-byte rows, fewer bank conflicts)

template <int NT>  // column tiles: 8 values of j each
__global__ __launch_bounds__(256) void k_adc_product(DirectAdcArgs a, LinSamples l) {
    __shared__ __attribute__((aligned(16))) float val[4][2][kProdChunk][kProdPad];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 15, kq = lane >> 4;
    const int half = lane >> 5, mb = lane & 31;
    const int64_t K = a.K;
    const int coil = blockIdx.y;
    const float *sre = a.coil_re ? a.coil_re + (int64_t)coil * K : nullptr;
    const float *sim = a.coil_im ? a.coil_im + (int64_t)coil * K : nullptr;
    const double tau0 = half ? l.tau0 : 0.0, dtau = half ? 16.0 * l.dtau : l.dtau;
    cached_f32x4 d[2][NT];
    double acc[2][NT][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            d[r][c] = cached_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[r][c][v] = 0.0;
        }
    auto flush = [&](double gain0) {  // gain0: of the sums with A_0
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < NT; ++c) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[r][c][v] = r == 0 && v < 2 ? fma(gain0, (double)d[r][c][v], acc[r][c][v]) : acc[r][c][v] + (double)d[r][c][v];
                d[r][c] = cached_f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    const int64_t stride = (int64_t)gridDim.x * 4 * kProdChunk;
    int64_t base = ((int64_t)blockIdx.x * 4 + wave) * kProdChunk;
    // the next chunk's isochromats are loaded during this one's product
    float x = 0.f, y = 0.f, z = 0.f, df = 0.f, t2 = 1.f, cr = 1.f, ci = 0.f;
    double mx = 0.0, my = 0.0;
    auto load = [&](int64_t b) {
        const int64_t k = min(b + mb, K - 1);
        x = a.ph.x[k];
        y = a.ph.y[k];
        z = a.ph.z[k];
        df = a.ph.df[k];
        t2 = a.ph.t2[k];
        if (a.s64_in) {
            mx = a.s64_in[k];
            my = a.s64_in[K + k];
        } else if (a.min_x) {
            mx = a.min_x[k];
            my = a.min_y[k];
        }
        if (sre) {
            cr = sre[k];
            ci = sim[k];
        }
    };
    if (base < K) load(base);
    for (; base < K; base += stride) {
        const double step = fma(l.dc[0], (double)x, fma(l.dc[1], (double)y, fma(l.dc[2], (double)z, l.dtau * (double)df)));
        const double first = fma(l.c0[0], (double)x, fma(l.c0[1], (double)y, fma(l.c0[2], (double)z, l.tau0 * (double)df)));
        double p0 = half ? first - rint(first) : 0.0, dp = step - rint(step);
        if (half) {
            dp *= 16.0;
            dp -= rint(dp);
        }
        const double r2 = -kLog2e / (double)t2;
        const float e0 = (float)(tau0 * r2), de = (float)(dtau * r2);
        // pairs of other phases than 0, which is exact: B_j, A_1 .. A_15
        const bool turns = half && dp != 0.0;
        const double gain = 1.0 + kTurnBias * ((turns || p0 != 0.0) + turns);
        const int n_turns = __popcll(__ballot(turns));
        const double gain0 = kq == 0 ? 1.0 - kTurnBias / kProdChunk * n_turns : 1.0;  // A_0 is 1
        // the factor of every value of this side: 1 (A), or M S (B; 0 past the end)
        float wr = 1.f, wi = 0.f;
        if (half) {
            wr = base + mb < K ? (float)(mx * gain) : 0.f;
            wi = base + mb < K ? (float)(my * gain) : 0.f;
            if (sre) {
                const float t = wr * cr - wi * ci;
                wi = wr * ci + wi * cr;
                wr = t;
            }
        }
        float4 *out = (float4 *)val[wave][half][mb];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            float o[4];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float s, c;
                sincos_rev(fma((double)(e + q), dp, p0), &s, &c);
                const float g = __builtin_amdgcn_exp2f(fmaf((float)(e + q), de, e0));
                const float ur = g * wr, ui = g * wi;
                o[2 * q] = fmaf(ur, c, ui * s);  // (wr + i wi) g (c - i s)
                o[2 * q + 1] = fmaf(ui, c, -ur * s);
            }
            out[e / 2] = make_float4(o[0], o[1], o[2], o[3]);
        }
        if (base + stride < K) load(base + stride);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int t = 0; t < kProdChunk / 4; ++t) {
            const float *pa = val[wave][0][4 * t + kq], *pb = val[wave][1][4 * t + kq];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int c = 0; c < NT; ++c)
                    d[r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[16 * r + i], pb[16 * c + i], d[r][c], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        flush(gain0);
    }
    // Element v of tile (r, c): row 4 kq + v = {Re, Im} A_{8 r + 2 kq + v / 2}, column
    // i = {Re, Im} B_{8 c + i / 2}.  The neighbouring lane holds the other part of B.
    double2 *sum = (double2 *)val;  // [wave][sample]
    __syncthreads();
    const bool odd = lane & 1;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double re = acc[r][c][2 * u], im = acc[r][c][2 * u + 1];  // Re A x, Im A x (x: this lane's part of B)
                const double ore = dpp_f64<0xb1>(re), oim = dpp_f64<0xb1>(im);
                if (!odd)
                    sum[256 * wave + 8 * r + 2 * kq + u + 16 * (8 * c + (i >> 1))] = make_double2(re - oim, im + ore);
            }
    __syncthreads();
    for (int n = threadIdx.x; n < a.n_samples; n += 256) {
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            sr += sum[256 * w + n].x;
            si += sum[256 * w + n].y;
        }
        a.partial[((int64_t)coil * gridDim.x + blockIdx.x) * a.n_samples + n] = make_double2(sr, si);
    }
}

// Four workgroups per CU fill the chip; fewer partial sums than k_direct_adc's.
int adc_product_grid(int64_t K) {
    const int64_t blocks = (K + 4 * kProdChunk - 1) / (4 * kProdChunk);
    return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, 1024));
}

hipError_t launch_adc_product(const DirectAdcArgs &a, const LinSamples &l, int grid, hipStream_t st) {
    static_assert(sizeof(float) * 4 * 2 * kProdChunk * kProdPad >= sizeof(double2) * 4 * 256, "sums fit the values' LDS");
    if (a.n_samples < 1 || a.n_samples > 256 || grid < 1 || grid > kAdcMaxGrid || a.K < 1) return hipErrorInvalidValue;
    if (!a.coil_re != !a.coil_im || a.n_coils < 1 || a.n_coils > kMaxCoils) return hipErrorInvalidValue;
    const dim3 g((unsigned)grid, (unsigned)a.n_coils);
    if (a.n_samples <= 128)
        hipLaunchKernelGGL(k_adc_product<1>, g, dim3(256), 0, st, a, l);
    else
        hipLaunchKernelGGL(k_adc_product<2>, g, dim3(256), 0, st, a, l);
    return hipGetLastError();
}

hipError_t launch_cached(const CachedArgs &a, int mode, hipStream_t st) {
    const int64_t blocks = (a.K + kCachedBlock - 1) / kCachedBlock;
    if (blocks <= 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kCachedBlock);
    switch (mode) {
        case kCacheMap: hipLaunchKernelGGL(k_cached<kCacheMap>, grid, block, 0, st, a); break;
        case kCacheApply: hipLaunchKernelGGL(k_cached<kCacheApply>, grid, block, 0, st, a); break;
        case kCacheCompose: hipLaunchKernelGGL(k_cached<kCacheCompose>, grid, block, 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int direct_adc_grid(int64_t K) {
    const int64_t chunks = (K + kAdcBlock - 1) / kAdcBlock;
    return (int)(chunks < kAdcMaxGrid ? (chunks > 0 ? chunks : 1) : kAdcMaxGrid);
}

hipError_t launch_direct_adc(const DirectAdcArgs &a, int grid, hipStream_t st) {
    if (a.n_samples < 1 || a.n_samples > kAdcBlock || grid < 1 || grid > kAdcMaxGrid) return hipErrorInvalidValue;
    if (a.coil_re) {
        if (!a.coil_im || a.n_coils < 1 || a.n_coils > kMaxCoils) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_direct_adc<true>, dim3(grid), dim3(kAdcBlock), 0, st, a);
    } else {
        hipLaunchKernelGGL(k_direct_adc<false>, dim3(grid), dim3(kAdcBlock), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace gbs
