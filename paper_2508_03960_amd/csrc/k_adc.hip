// k_adc_lin: every ADC sample of a grouped with-ADC subsequence from the
// group sums (Eq. 8 with Eq. 10) when the sample times and moments are
// arithmetic in n (a constant readout gradient sampled at a fixed dwell).
// Then the factor of group g at sample n is a geometric sequence,
//     e^{-tau_n/T2} e^{-i phi_g(n)} = f_g z_g^n,
//     phi_g(n) = 2 pi (cyc_n x_g + df_g tau_n),
// so a thread evaluates f_g z_g^{n0} directly (FP64 phase reduced modulo one
// turn, hardware sin/cos), steps 15 further samples by complex multiplication
// with z_g, restarts at n0 + 16 from f_g z_g^{n0} times z_g^16 (itself made
// directly, not by repeated products) and steps 15 more.  The FP32 rounding
// of z_g thus compounds over at most 15 products.
// The workgroup first stages what its groups need in LDS: coordinate, df and
// the group sum, and z_g, z_g^16 and 1/T2, made once per group.  The group
// loop then touches no global memory, so its pace does not depend on the
// memory latency (the final-state gather runs beside it).
// Thread layout: 32 consecutive samples per thread ("chunk"), threads with the
// same chunk split the workgroup's groups ("slices").  A thread adds its
// groups' terms (at most kAdcLinGroups / slices, 28 for a 256-sample
// readout) in FP32, the terms themselves being FP32 products; the eight
// slices of a wavefront that share a chunk add in FP32 through lane shuffles;
// those sums go through LDS, and the workgroup's rows and the workgroups add
// in FP64 (one FP64 atomic pair per sample and workgroup).
//
// k_adc_mm: the same for many readouts of equal timing at once, as a matrix
// product (below).  k_adc_lin takes what is left: readouts that would fill too
// little of a tile (adc_mm_min_rows), timings with few terms, and calls whose
// workspace has no room for the product's partial sums.
#include "adc.hpp"
#include "device_math.hpp"

namespace gbs {

constexpr int kAdcLinWG = 256;
constexpr int kAdcLinChunk = 32;      // samples per thread
constexpr int kAdcLinGroups = 896;    // groups per workgroup: 40 KiB of LDS, 4 workgroups per CU
constexpr int kAdcLinHalf = kAdcLinChunk / 2;

// Group-table rows and group sums through the global address space (the
// pointers come out of the job descriptor and would otherwise be flat loads).
typedef const __attribute__((address_space(1))) float *adc_gf32;
typedef const __attribute__((address_space(1))) double *adc_gf64;
__device__ __forceinline__ float4 adc_row(const float4 *tab, int g) {
    adc_gf32 p = (adc_gf32)(tab + g);
    return make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ double2 adc_sum(const double2 *gs, int g) {
    adc_gf64 p = (adc_gf64)(gs + g);
    return make_double2(p[0], p[1]);
}

__global__ __launch_bounds__(kAdcLinWG) void k_adc_lin(const AdcLinJob *__restrict__ jobs, double *__restrict__ sig_base) {
    // [slice / 8][sample]: the eight-slice sums (8 KiB); per group of the
    // workgroup (coord, df, Re S, Im S), (z, z^16) and 1/T2 (31.5 KiB)
    __shared__ float2 red[kAdcLinWG * kAdcLinChunk / 8];
    __shared__ float4 ga[kAdcLinGroups];
    __shared__ float4 gb[kAdcLinGroups];
    __shared__ float gr[kAdcLinGroups];
    const AdcLinJob j = jobs[blockIdx.y];
    const int g0 = blockIdx.x * kAdcLinGroups;
    if (g0 >= j.n_groups) return;  // uniform over the workgroup
    const int ng = min(kAdcLinGroups, j.n_groups - g0);
    double *sig = sig_base + 2 * j.sig_offset;
    // all loads first (indices clamped into the workgroup's groups), then the
    // arithmetic and the LDS writes of the groups that exist
    constexpr int kRounds = (kAdcLinGroups + kAdcLinWG - 1) / kAdcLinWG;
    float4 pr[kRounds];
    double2 Sr[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = min((int)threadIdx.x + r * kAdcLinWG, ng - 1);
        pr[r] = adc_row(j.gtab, g0 + i);  // (coord, T1, T2, df)
        Sr[r] = adc_sum(j.gsum, g0 + i);
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = threadIdx.x + r * kAdcLinWG;
        if (i < ng) {
            const float4 p = pr[r];
            const double2 S = Sr[r];
            const double dphi = j.dcyc * (double)p.x + (double)p.w * j.dtau;  // turns per sample
            float sd, cd, sh, ch;
            sincos_rev(dphi, &sd, &cd);
            sincos_rev(kAdcLinHalf * dphi, &sh, &ch);
            const float r2 = __builtin_amdgcn_rcpf(p.z);
            const float ed = __expf(-(float)j.dtau * r2), eh = __expf(-(float)(kAdcLinHalf * j.dtau) * r2);
            ga[i] = make_float4(p.x, p.w, (float)S.x, (float)S.y);
            gb[i] = make_float4(ed * cd, -ed * sd, eh * ch, -eh * sh);  // z = ed e^{-i dphi}, z^16
            gr[i] = r2;
        }
    }
    __syncthreads();
    // chunks per pass: power of two covering the samples, at most 8, so
    // that 8 slices sharing a chunk sit in one wavefront
    int n_chunks = 1;
    while (n_chunks < kAdcLinWG / kAdcLinChunk && n_chunks * kAdcLinChunk < j.n_samples) n_chunks <<= 1;
    const int n_slices = kAdcLinWG / n_chunks;
    const int chunk = threadIdx.x % n_chunks, slice = threadIdx.x / n_chunks;
    const int per_pass = n_chunks * kAdcLinChunk;
    for (int base = 0; base < j.n_samples; base += per_pass) {
        const int n0 = base + chunk * kAdcLinChunk;
        const int cnt = max(0, min(kAdcLinChunk, j.n_samples - n0));
        const double tau_n0 = j.tau0 + n0 * j.dtau, cyc_n0 = j.cyc0 + n0 * j.dcyc;
        const float mtau_n0 = -(float)tau_n0;
        float ar[kAdcLinChunk], ai[kAdcLinChunk];
#pragma unroll
        for (int k = 0; k < kAdcLinChunk; ++k) ar[k] = ai[k] = 0.f;
        if (cnt > 0 && slice < ng) {
            // the next group's rows are read one iteration ahead
            float4 a_next = ga[slice], b_next = gb[slice];
            float r2_next = gr[slice];
            for (int i = slice; i < ng; i += n_slices) {
                const float4 a = a_next, b = b_next;
                const float r2 = r2_next;
                if (i + n_slices < ng) {
                    a_next = ga[i + n_slices];
                    b_next = gb[i + n_slices];
                    r2_next = gr[i + n_slices];
                }
                float s0, c0;
                sincos_rev(cyc_n0 * (double)a.x + (double)a.y * tau_n0, &s0, &c0);
                const float e0 = __expf(mtau_n0 * r2);
                // f = S e0 e^{-i phi(n0)}
                const float tr = e0 * c0, ti = -e0 * s0;
                const float f0r = a.z * tr - a.w * ti;
                const float f0i = a.z * ti + a.w * tr;
                float fr = f0r, fi = f0i;
#pragma unroll
                for (int k = 0; k < kAdcLinHalf; ++k) {
                    ar[k] += fr;
                    ai[k] += fi;
                    const float nr = fr * b.x - fi * b.y;
                    fi = fr * b.y + fi * b.x;
                    fr = nr;
                }
                fr = f0r * b.z - f0i * b.w;  // f_g z_g^{n0 + 16}: f_g z_g^{n0} times z_g^16
                fi = f0r * b.w + f0i * b.z;
#pragma unroll
                for (int k = kAdcLinHalf; k < kAdcLinChunk; ++k) {
                    ar[k] += fr;
                    ai[k] += fi;
                    const float nr = fr * b.x - fi * b.y;
                    fi = fr * b.y + fi * b.x;
                    fr = nr;
                }
            }
        }
        // lanes l ^ (m n_chunks), m < 8: one chunk, eight slices of a
        // wavefront; the slices that are multiples of 8 then hold the sums and
        // write them, one row each.  Four samples at a time: the scheduling
        // barrier keeps the compiler from putting every shuffle in flight at
        // once, which would take as many registers again as the sums.
        const int rows = n_slices / 8;
        const bool leader = slice % 8 == 0;
        float2 *mine = red + (slice / 8) * per_pass + chunk * kAdcLinChunk;
#pragma unroll
        for (int k0 = 0; k0 < kAdcLinChunk; k0 += 4) {
#pragma unroll
            for (int m = 1; m < 8; m <<= 1) {
#pragma unroll
                for (int k = k0; k < k0 + 4; ++k) {
                    ar[k] += __shfl_xor(ar[k], m * n_chunks);
                    ai[k] += __shfl_xor(ai[k], m * n_chunks);
                }
            }
            if (leader) {
#pragma unroll
                for (int k = k0; k < k0 + 4; ++k) mine[k] = make_float2(ar[k], ai[k]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        for (int n = threadIdx.x; n < per_pass; n += kAdcLinWG) {
            if (base + n < j.n_samples) {
                double sr = 0.0, si = 0.0;
                for (int r = 0; r < rows; ++r) {
                    const float2 v = red[r * per_pass + n];
                    sr += (double)v.x;
                    si += (double)v.y;
                }
                atomicAdd(&sig[2 * (base + n)], sr);
                atomicAdd(&sig[2 * (base + n) + 1], si);
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- k_adc_mm
// A workgroup takes 64 readouts of one class, 128 samples and up to 224 groups:
// A = the readouts' group sums (rounded to FP32, staged 32 groups at a time),
// B = e^{-tau_n/T2} e^{-i phi_g(n)}, evaluated directly per (group, sample) in
// the lanes that hold it, four real v_mfma_f32_16x16x4_f32 per complex 16 x 16
// tile and four groups.  A wavefront holds all 64 rows of its 32 samples, so
// each factor is made once per 64 readouts: VALU work is a fifth of the matrix
// core's, which bounds the kernel.  The 32 groups of a stage add in the matrix
// core, the stages in FP32 (up to seven), FP64 from there (k_adc_mm_sum); no
// atomics.  (All 224 groups in the matrix core's FP32 sums erred by 6.0e-7 of the
// signal for equal terms of 100000 groups, where k_adc_lin errs by 3.0e-7; this
// by 2.3e-7, in the same time.)
typedef float adc_f32x4 __attribute__((ext_vector_type(4)));

struct AdcGroup {
    double x, df;
};

__global__ __launch_bounds__(256, 2) void k_adc_mm(const AdcClass *__restrict__ classes, const AdcRow *__restrict__ rows,
                                                const AdcTile *__restrict__ tiles, float2 *__restrict__ part) {
    constexpr int ET = kAdcMmRows / 16, NT = kAdcMmCols / 64, RQ = kAdcMmRows / 8;
    constexpr int LD = kAdcMmSub + 4;
    __shared__ float2 sA[kAdcMmRows * LD];
    __shared__ AdcGroup sg[kAdcMmSub];
    __shared__ float sr2[kAdcMmSub];
    const AdcTile tl = tiles[blockIdx.y];
    const AdcClass c = classes[tl.cls];
    const int g0 = blockIdx.x * c.split;
    if ((int)blockIdx.x >= c.n_split) return;  // uniform
    const int g1 = min(g0 + c.split, c.n_groups);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 15, kq = lane >> 4;
    // staging: thread t loads group t % 32 of the rows t / 32 + 8 q
    const int sgp = threadIdx.x & 31, srow = threadIdx.x >> 5;
    const double2 *src[RQ];
#pragma unroll
    for (int q = 0; q < RQ; ++q) src[q] = rows[tl.row + min(srow + 8 * q, tl.n_rows - 1)].gsum;
    double2 sv[RQ];
    float4 gv = make_float4(0.f, 1.f, 1.f, 0.f);
    auto load = [&](int g) {  // groups g .. g + 31 (indices clamped; groups past the end are zeroed when stored)
        const int k = min(g + sgp, g1 - 1);
#pragma unroll
        for (int q = 0; q < RQ; ++q) sv[q] = adc_sum(src[q], k);
        if (threadIdx.x < kAdcMmSub) gv = adc_row(c.gtab, k);
    };
    double cyc[NT], tau[NT];
    float mtau[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = tl.n0 + 16 * (NT * wave + t) + i;
        tau[t] = c.tau0 + n * c.dtau;
        cyc[t] = c.cyc0 + n * c.dcyc;
        mtau[t] = -(float)tau[t];
    }
    adc_f32x4 tr[ET][NT], ti[ET][NT];
#pragma unroll
    for (int e = 0; e < ET; ++e)
#pragma unroll
        for (int t = 0; t < NT; ++t) tr[e][t] = ti[e][t] = adc_f32x4{0.f, 0.f, 0.f, 0.f};
    const bool live = tl.n0 + 16 * NT * wave < c.n_samples;
    load(g0);
    for (int g = g0; g < g1; g += kAdcMmSub) {
        __syncthreads();  // the previous groups have been read
        const bool in = g + sgp < g1;
#pragma unroll
        for (int q = 0; q < RQ; ++q)
            sA[(srow + 8 * q) * LD + sgp] = in ? make_float2((float)sv[q].x, (float)sv[q].y) : make_float2(0.f, 0.f);
        if (threadIdx.x < kAdcMmSub) {
            sg[threadIdx.x] = AdcGroup{(double)gv.x, (double)gv.w};
            sr2[threadIdx.x] = __builtin_amdgcn_rcpf(gv.z);
        }
        __syncthreads();
        if (g + kAdcMmSub < g1) load(g + kAdcMmSub);
        if (!live) continue;
        adc_f32x4 dr[ET][NT], di[ET][NT];
#pragma unroll
        for (int e = 0; e < ET; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) dr[e][t] = di[e][t] = adc_f32x4{0.f, 0.f, 0.f, 0.f};
        const int steps = (min(kAdcMmSub, g1 - g) + 3) / 4;
        for (int s = 0; s < steps; ++s) {
            const AdcGroup p = sg[4 * s + kq];
            const float r2 = sr2[4 * s + kq];
            float fr[NT], fi[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float sn, co;
                sincos_rev(cyc[t] * p.x + p.df * tau[t], &sn, &co);
                const float e = __expf(mtau[t] * r2);
                fr[t] = e * co;
                fi[t] = -e * sn;
            }
#pragma unroll
            for (int e = 0; e < ET; ++e) {
                const float2 a = sA[(16 * e + i) * LD + 4 * s + kq];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    dr[e][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, fr[t], dr[e][t], 0, 0, 0);
                    di[e][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, fi[t], di[e][t], 0, 0, 0);
                    dr[e][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, -fi[t], dr[e][t], 0, 0, 0);
                    di[e][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, fr[t], di[e][t], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < ET; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                tr[e][t] += dr[e][t];
                ti[e][t] += di[e][t];
            }
    }
    if (!live) return;
    // element v of a tile: row 4 kq + v, column i
#pragma unroll
    for (int e = 0; e < ET; ++e)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * e + 4 * kq + v;
            if (r >= tl.n_rows) continue;
            const AdcRow &row = rows[tl.row + r];
            float2 *o = part + row.part + blockIdx.x * row.stride;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int n = tl.n0 + 16 * (NT * wave + t) + i;
                if (n < c.n_samples) o[n] = make_float2(tr[e][t][v], ti[e][t][v]);
            }
        }
}

// sig += the splits' partial sums, FP64: 64 samples per workgroup, wavefront w
// of 16 adding the splits w, w + 16, ... in order, then the 16 sums in order
// (few rows with many splits are a chain of loads; four wavefronts took twice
// as long for 128 rows of 290 splits).
constexpr int kAdcSumWaves = 16;
__global__ __launch_bounds__(64 * kAdcSumWaves) void k_adc_mm_sum(const AdcClass *__restrict__ classes, const AdcRow *__restrict__ rows,
                                                    const float2 *__restrict__ part, double *__restrict__ sig) {
    __shared__ double2 red[kAdcSumWaves][64];
    const AdcRow r = rows[blockIdx.x];
    const int ns = classes[r.cls].n_samples, n_split = classes[r.cls].n_split;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = blockIdx.y * 64 + lane;
    if ((int)blockIdx.y * 64 >= ns) return;  // uniform
    const float2 *p = part + r.part + min(n, ns - 1);
    double sr = 0.0, si = 0.0;
    int s = wave;
    constexpr int W = kAdcSumWaves;
    for (; s + 3 * W < n_split; s += 4 * W) {  // four loads in flight
        float2 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = p[(s + W * q) * r.stride];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sr += v[q].x;
            si += v[q].y;
        }
    }
    for (; s < n_split; s += W) {
        const float2 v = p[s * r.stride];
        sr += v.x;
        si += v.y;
    }
    red[wave][lane] = make_double2(sr, si);
    __syncthreads();
    if (wave == 0 && n < ns) {
        sr = si = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sr += red[w][lane].x;
            si += red[w][lane].y;
        }
        double *o = sig + 2 * (r.sig_offset + n);
        o[0] += sr;
        o[1] += si;
    }
}

hipError_t launch_adc_mm(const AdcClass *cls, const AdcRow *rows, const AdcTile *tiles, const AdcBatch &b, float2 *part,
                         double *sig, hipStream_t st) {
    if (b.n_tiles <= 0) return hipSuccess;
    if (b.n_tiles > 65535 || b.max_samples > 64 * 65535 || b.max_split <= 0 || b.n_rows <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_adc_mm, dim3((unsigned)b.max_split, (unsigned)b.n_tiles), dim3(256), 0, st, cls, rows,
                       tiles + b.tile0, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_adc_mm_sum, dim3((unsigned)b.n_rows, (unsigned)((b.max_samples + 63) / 64)),
                       dim3(64 * kAdcSumWaves), 0, st, cls, rows + b.row0, part, sig);
    return hipGetLastError();
}

hipError_t launch_adc_lin(const AdcLinJob *jobs, int n_jobs, int max_groups, double *sig, hipStream_t st) {
    if (n_jobs <= 0 || max_groups <= 0) return hipSuccess;
    dim3 grid((max_groups + kAdcLinGroups - 1) / kAdcLinGroups, n_jobs);
    hipLaunchKernelGGL(k_adc_lin, grid, dim3(kAdcLinWG), 0, st, jobs, sig);
    return hipGetLastError();
}

}  // namespace gbs
