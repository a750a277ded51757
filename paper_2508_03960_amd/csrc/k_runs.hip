// Grouped simulation per run of the layout on gfx950 (see runs.hpp).
//
//  k_run_y      Y_r(c) of every run and y moment c on an even grid, as a matrix
//               product over the members: a line's phase is the product of one
//               of 8 a-phases and one of 8 b-phases per 256 lines,
//                 c = c0 + d (+-(i + 1/2) +- (16 j + 8)),
//               so per member 16 rows {cos, sin}(a_i y) and 16 columns
//               {cos, sin}(b_j y), weighted by the real and by the imaginary
//               part of the member's weight, give all 256 lines (both signs
//               share the four real products): two v_mfma_f32_16x16x4_f32 per
//               four members, 4 flops per member and line.
//  k_run_sweep  all operations of a simulation with one run per lane.
//  k_run_state  the final state in the caller's order from the runs' ratios.
#include <type_traits>

#include "device_math.hpp"
#include "kernels.hpp"
#include "runs.hpp"
#include "sweep_math.hpp"

namespace gbs {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- k_run_y
// One workgroup per kRunTile runs (a row of the Y layout), which its four
// wavefronts take one after the other.  A wavefront takes a run's members 32 at a
// time.  Lane l first makes the eight a-phases (l < 32) or b-phases (l >= 32) of
// member l % 32: the first one, the step and four steps directly (v_sin / v_cos take turns), the others by at
// most four products of those, and the weight with the phase of c0; all of it
// goes to LDS.  Then every step of the product reads four members, lane l
// holding row l % 16 and column l % 16 of member l / 16.  Evaluated in the lanes
// of the product instead, the 32 phases of a member took 95 VALU cycles per
// step, against 64 of the matrix core (27.3M members, 256 lines: 555 us).
// The matrix core adds the members of one chunk, the chunks' sums add in FP32
// eight at a time, and those in FP64: 2.4e-7 of the signal off at any length.
// All of a run's members in one FP32 accumulator were 1.4e-4 off at 16384 equal
// terms and 9e-3 at 2^20, measurably from 64 on; that took 4 to 6 % less time
// (27.3M isochromats: 256 lines 524 and 554 us, 128 lines 348 and 360).
// A phase coefficient (turns per metre) as two floats: c y mod 1 then takes
// four FP32 instructions with one rounding of the reduced phase (the FMA of
// hi y - rint(hi y) is exact up to it), instead of five at FP64.
struct Coef {
    float hi, lo;
};
__device__ __forceinline__ Coef coef_of(double c) {
    const float h = (float)c;
    return Coef{h, (float)(c - (double)h)};
}
__device__ __forceinline__ float turns(const Coef &c, float y) {
    return fmaf(c.lo, y, fmaf(c.hi, y, -rintf(c.hi * y)));
}

__device__ __forceinline__ float2 phase_at(const Coef &c, float y) {  // (cos, sin)
    const float t = turns(c, y);
    return make_float2(__builtin_amdgcn_cosf(t), __builtin_amdgcn_sinf(t));
}
__device__ __forceinline__ float2 turned(const float2 &p, const float2 &q) {
    return make_float2(fmaf(p.x, q.x, -p.y * q.y), fmaf(p.x, q.y, p.y * q.x));
}

// V_SIN/V_COS pairs in phase e of a member (the first, the step, four steps)
__device__ __forceinline__ int factors_of(int e) { return 1 + (e & 3) + (e >> 2); }

constexpr int kRunChunk = 32;
constexpr int kRunFlush = 8;  // chunks whose sums add in FP32

// HALF: at most 128 lines (b-phases 0 .. 3), columns 0 .. 7 with the real and
// 8 .. 15 with the imaginary part of the weight: one matrix instruction per step.
template <bool COILS, bool HALF>
__global__ __launch_bounds__(256) void k_run_y(RunYArgs a) {
    // {cos, sin} of the a, of the b; the four float4 of member k in the order
    // e ^ (k / 4 % 4): writes and reads are free of bank conflicts without
    // padding.  With that and the tile of the lines that are made, HALF takes 26
    // KB and six workgroups fit a CU instead of four (27.3M members, 128 lines:
    // 373 -> 348 us when that was done; 36 KB and four as before for 256 lines).
    __shared__ __attribute__((aligned(16))) float phases[4][2][kRunChunk][16];
    __shared__ float2 weight[4][kRunChunk];
    constexpr int l0 = HALF ? 64 : 0, l1 = HALF ? 192 : kRunLinesSet;  // the set's lines that are made
    __shared__ float2 tile[l1 - l0][kRunTile + 1];  // + 1: the lines of a store fall into different banks
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int set = blockIdx.y % ((a.lines.nb + 7) / 8), coil = blockIdx.y / ((a.lines.nb + 7) / 8);
    const int i = lane & 15, kq = lane >> 4;
    const int half = lane >> 5, mb = lane & 31;  // the lane's share of the phases
    const Coef f0 = coef_of((half ? 128 * set + 8 : 0.5) * a.lines.d), f1 = coef_of((half ? 16 : 1) * a.lines.d),
               f4 = coef_of((half ? 64 : 4) * a.lines.d), c0 = coef_of(a.lines.c0);
    const int64_t tile0 = a.r0 + (int64_t)blockIdx.x * kRunTile;  // first run of the workgroup
    const int64_t rend = a.r0 + a.n;
    // slots relative to the workgroup's first one (32 bits: the layout has at most kRunMaxSlots)
    const int64_t slot0 = 4 * (int64_t)a.first4[tile0];
    const int last = (int)(4 * (int64_t)a.first4[a.n_runs] - 1 - slot0);
    const float *y = a.y + slot0, *m0 = a.m0 + slot0;
    const float *sre = COILS ? a.coil + 2 * coil * a.coil_plane + slot0 : nullptr;
    const float *sim = COILS ? sre + a.coil_plane : nullptr;
    int slot = 0;
    float yv = 0.f, mv = 0.f, cr = 1.f, ci = 0.f;
    auto fetch = [&](int base) {  // members of the next slots (the layout's last slot past its end)
        slot = base + mb;
        const uint32_t s = 4u * (uint32_t)min(slot, last);
        yv = *at_bytes(y, s);
        mv = *at_bytes(m0, s);
        if (COILS) {
            cr = *at_bytes(sre, s);
            ci = *at_bytes(sim, s);
        }
    };
    auto first_slot = [&](int64_t r) { return (int)(4 * (int64_t)a.first4[r] - slot0); };
    // The wavefronts take the workgroup's runs one by one (the lengths differ
    // widely: with fixed shares the longest held the others up).  A run is
    // taken before the one ahead of it is summed, so its first members are
    // loaded in time.
    __shared__ int taken;
    __shared__ float2 still[4];  // the weights of a run's members at y = 0
    if (threadIdx.x == 0) taken = 4;
    __syncthreads();
    int j = wave;
    if (tile0 + j < rend) fetch(first_slot(tile0 + j));
    while (j < kRunTile) {
        int nj = 0;
        if (lane == 0) nj = atomicAdd(&taken, 1);
        nj = __builtin_amdgcn_readfirstlane(nj);
        const int64_t r = tile0 + j, rn = tile0 + nj;
        const int next = nj < kRunTile && rn < rend ? first_slot(rn) : last;
        f32x4 dr = {0.f, 0.f, 0.f, 0.f}, di = {0.f, 0.f, 0.f, 0.f};
        bool any_still = false;
        if (r < rend) {
            const int s0 = first_slot(r), s1 = first_slot(r + 1);
            f32x4 tr = dr, ti = di;
            double ar[4] = {0.0, 0.0, 0.0, 0.0}, ai[4] = {0.0, 0.0, 0.0, 0.0};
            for (int base = s0; base < s1; base += kRunChunk) {
                float2 p[8];
                p[0] = phase_at(f0, yv);
                const float2 q1 = phase_at(f1, yv), q4 = phase_at(f4, yv), w = phase_at(c0, yv);
#pragma unroll
                for (int e = 1; e < 4; ++e) p[e] = turned(p[e - 1], q1);
#pragma unroll
                for (int e = 4; e < 8; ++e) p[e] = turned(p[e - 4], q4);
                const float m = slot < s1 ? mv : 0.f;
                float2 v;  // m0 S(k, p) e^{-i phi}
                if (COILS) {
                    const float pr = m * cr, pi = m * ci;
                    v = make_float2(fmaf(pr, w.x, pi * w.y), fmaf(pi, w.x, -pr * w.y));
                } else {
                    v = make_float2(m * w.x, -m * w.y);
                }
                if (__ballot(yv == 0.f && m != 0.f)) {
                    const bool at0 = yv == 0.f && !half;
                    const float sx = wave_sum_lane63(at0 ? v.x : 0.f), sy = wave_sum_lane63(at0 ? v.y : 0.f);
                    if (lane == 63) {
                        const float2 o = any_still ? still[wave] : make_float2(0.f, 0.f);
                        still[wave] = make_float2(o.x + sx, o.y + sy);
                    }
                    any_still = true;
                }
                float4 *ph = (float4 *)phases[wave][half][mb];
#pragma unroll
                for (int e = 0; e < 4; ++e) ph[e ^ (mb >> 2 & 3)] = make_float4(p[2 * e].x, p[2 * e].y, p[2 * e + 1].x, p[2 * e + 1].y);
                if (!half) weight[wave][mb] = v;
                const int left = s1 - base;
                fetch(left > kRunChunk ? base + kRunChunk : next);
                const int steps = min(left, kRunChunk) / 4;
                if (base > s0) {
                    tr += dr;
                    ti += di;
                    dr = di = f32x4{0.f, 0.f, 0.f, 0.f};
                    if ((base - s0) % (kRunFlush * kRunChunk) == 0) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            ar[v] += (double)tr[v];
                            if (!HALF) ai[v] += (double)ti[v];
                        }
                        tr = ti = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (int t = 0; t < steps; t += 4) {  // (members past the run's end have weight 0)
                    float pa[4], pb[4];
                    float2 pw[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int k = 4 * (t + e) + kq;
                        pa[e] = phases[wave][0][k][i ^ 4 * e];
                        pb[e] = phases[wave][1][k][(HALF ? i & 7 : i) ^ 4 * e];
                        if (HALF)
                            pw[e].x = ((const float *)&weight[wave][k])[i >> 3];
                        else
                            pw[e] = weight[wave][k];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dr = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[e], pb[e] * pw[e].x, dr, 0, 0, 0);
                        if (!HALF) di = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[e], pb[e] * pw[e].y, di, 0, 0, 0);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            dr += tr;
            di += ti;
            if (s1 - s0 > kRunFlush * kRunChunk) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    dr[v] = (float)(ar[v] + (double)dr[v]);
                    if (!HALF) di[v] = (float)(ai[v] + (double)di[v]);
                }
            }
        }
        // lane (column 2 jb + t, rows 4 kq ..): element v of the tiles is
        // {cos, sin}(a_{2 kq + v / 2}) times {cos, sin}(b_jb); neighbouring
        // lanes trade halves, then lane parity picks the a index
        if (HALF) {  // the other weight's sums from the lane eight columns away
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float o = dpp_f32<0x128>(dr[v]);  // row_ror:8
                di[v] = i < 8 ? o : dr[v];
                dr[v] = i < 8 ? dr[v] : o;
            }
        }
        const bool odd = lane & 1;
        auto trade = [&](const f32x4 &v, float &cc, float &sc, float &cs, float &ss) {
            const float g0 = dpp_f32<0xb1>(odd ? v[0] : v[2]), g1 = dpp_f32<0xb1>(odd ? v[1] : v[3]);
            cc = odd ? g0 : v[0];
            sc = odd ? g1 : v[1];
            cs = odd ? v[2] : g0;
            ss = odd ? v[3] : g1;
        };
        float rcc, rsc, rcs, rss, icc, isc, ics, iss;
        trade(dr, rcc, rsc, rcs, rss);
        trade(di, icc, isc, ics, iss);
        const int ia = 2 * kq + (lane & 1), jb = HALF ? (i & 7) >> 1 : i >> 1;
        const float gain = (float)(kTurnBias * ((a.lines.d != 0.0 ? factors_of(ia) + factors_of(jb) : 0) + (a.lines.c0 != 0.0)));
        // (phases of members at y = 0 are exact: they get no gain)
        const float2 w0 = any_still ? still[wave] : make_float2(0.f, 0.f);
        // sum (wr + i wi)(cos t - i sin t), t = sa a + sb b
        auto put = [&](int line, float sa, float sb) {
            const float wrc = fmaf(-sa * sb, rss, rcc), wrs = fmaf(sa, rsc, sb * rcs);
            const float wic = fmaf(-sa * sb, iss, icc), wis = fmaf(sa, isc, sb * ics);
            const float re = wrc + wis, im = wic - wrs;
            tile[line - l0][j] = make_float2(fmaf(re - w0.x, gain, re), fmaf(im - w0.y, gain, im));
        };
        // lines 0 .. 127: -b of the set (descending), 128 .. 255: +b
        // (HALF: a line from one of the two lanes that hold its sums)
        if (!HALF || i < 8) {
            put(128 + 16 * jb + 8 + ia, 1.f, 1.f);
            put(128 + 16 * jb + 7 - ia, -1.f, 1.f);
        }
        if (!HALF || i >= 8) {
            put(128 - 16 * jb - 8 + ia, 1.f, -1.f);
            put(128 - 16 * jb - 9 - ia, -1.f, -1.f);
        }
        j = nj;
    }
    __syncthreads();
    const int mid = 16 * a.lines.nb, n_lines = a.lines.n_lines;
    float2 *out = a.out + coil * a.out_coil + ((int64_t)blockIdx.x * n_lines) * kRunTile;
    for (int e = l0 * kRunTile + threadIdx.x; e < l1 * kRunTile; e += 256) {
        const int ll = e / kRunTile, rr = e % kRunTile;
        const int line = ll < 128 ? mid - 128 * (set + 1) + ll : mid + 128 * set + (ll - 128);
        if (line >= 0 && line < n_lines) out[(int64_t)line * kRunTile + rr] = tile[ll - l0][rr];
    }
}

hipError_t launch_run_y(const RunYArgs &a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    if (a.lines.nb < 1 || a.lines.n_lines != 32 * a.lines.nb || a.r0 % kRunTile) return hipErrorInvalidValue;
    const int64_t tiles = (a.n + kRunTile - 1) / kRunTile;
    const int64_t gy = (int64_t)((a.lines.nb + 7) / 8) * a.n_coils;
    if (tiles > 0x7fffffff || gy > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles, (unsigned)gy);
    const bool half = a.lines.nb <= 4;
    if (a.coil && half)
        hipLaunchKernelGGL((k_run_y<true, true>), grid, dim3(256), 0, st, a);
    else if (a.coil)
        hipLaunchKernelGGL((k_run_y<true, false>), grid, dim3(256), 0, st, a);
    else if (half)
        hipLaunchKernelGGL((k_run_y<false, true>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_run_y<false, false>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

// ------------------------------------------------------------- k_run_sweep
// One run per lane, one wavefront per workgroup.  Every load of an operation
// depends on its descriptor and the lane's groups alone, and every operation
// of a part of the list issues the same loads in the same order: so the rows
// of the next kDepth operations are in flight during this one's arithmetic, and
// the wait for one operation's rows counts the later loads off instead of
// draining them (Y comes from HBM, a microsecond or two away).  The group sums
// of an emission are a segmented scan over the lanes (the runs of an x-group
// are neighbours): six DPP steps with the lane's masks, made once.  Wavefronts
// take whole x-groups, so a group's sum is one store; only a group of more than
// 64 runs adds its parts with atomics to the cleared sum (FP64 atomics of two
// neighbours per wavefront and emission made the sweep three times slower).
template <int CTRL>
__device__ __forceinline__ void seg_add(float mask, float &v) {
    v = fmaf(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true)), mask, v);
}

template <int MC>
__global__ __launch_bounds__(64) void k_run_sweep(RunSweepArgs a) {
    const int lane = threadIdx.x;
    const int64_t w0 = a.first[blockIdx.x], w1 = a.first[blockIdx.x + 1];
    const bool act = w0 + lane < w1;
    const int64_t r = act ? w0 + lane : w1 - 1;
    const int64_t rl = r - a.r0;
    const int gx = a.gx[r], gz = a.gz[r];
    const int key = act ? gx : -1;
    // masks of the segmented scan
    auto mask_of = [&](bool has, int src) {
        const int k = __shfl(key, src & 63);  // (by every lane, also those without a source)
        return has && k == key ? 1.f : 0.f;
    };
    const int row = lane >> 4;
    const float m1 = mask_of((lane & 15) >= 1, lane - 1), m2 = mask_of((lane & 15) >= 2, lane - 2);
    const float m4 = mask_of((lane & 15) >= 4, lane - 4), m8 = mask_of((lane & 15) >= 8, lane - 8);
    const float mb15 = mask_of(row & 1, 16 * row - 1), mb31 = mask_of(row >= 2, 31);
    const int knext = __shfl_down(key, 1);
    const bool end = act && (lane == 63 || knext != key);
    // does the x-group go on before or after the wavefront's runs?
    const bool own = key != (w0 > 0 ? a.gx[w0 - 1] : -1) && key != (w1 < a.n_runs ? a.gx[w1] : -1);
    // byte offsets (32 bits: checked at the launch); lanes of a wavefront lie in
    // at most 64 / kRunTile + 1 tiles of Y from its first one on
    const int64_t t0 = (w0 - a.r0) / kRunTile;
    const int coil0 = MC * (int)blockIdx.y;  // the wavefront's coils
    const float2 *yb = a.y + coil0 * a.y_coil + t0 * (int64_t)a.n_lines * kRunTile;
    const uint32_t oy = (uint32_t)(8 * ((rl / kRunTile - t0) * (int64_t)a.n_lines * kRunTile + rl % kRunTile));
    const uint32_t ox = 16u * (uint32_t)gx, oz = 8u * (uint32_t)gz;
    const uint32_t otx = 48u * (uint32_t)gx, otz = 48u * (uint32_t)gz, otr = 48u * (uint32_t)r;

    const int n_coils = min(a.n_coils - coil0, MC);
    const int64_t y_coil = a.y_coil;
    struct Meta {  // of an operation whose rows are in flight
        int flags, stride;
        double2 *gsum;
    };
    struct Rows {
        float4 px, t0, t1, t2;
        float2 pz, ex, ez, y[MC];
    };
    auto fetch_emit = [&](const RunOp &op, Rows &d) {
        d.ex = gather_at((const float2 *)op.emit_xtab, (op.flags & kOpEmit) ? ox : 0u);
        d.ez = gather_at(op.emit_ztab, (op.flags & kRunEmitZ) ? oz : 0u);
#pragma unroll
        for (int p = 0; p < MC; ++p)
            d.y[p] = gather_at(yb + min(p, n_coils - 1) * y_coil + op.line * kRunTile, oy);
    };
    auto fetch_full = [&](const RunOp &op, Rows &d) {
        d.px = gather_at(op.pre_xtab, (op.flags & kRunPreX) ? ox : 0u);
        d.pz = gather_at(op.pre_ztab, (op.flags & kRunPreZ) ? oz : 0u);
        // (the asm makes them values: a choice between the captured variables
        // themselves would go through memory)
        uint32_t o0 = otx, o2 = otz, o3 = otr;
        asm("" : "+v"(o0), "+v"(o2), "+v"(o3));
        uint32_t ot = op.rf_axis == 0 ? o0 : op.rf_axis == 2 ? o2 : o3;
        ot = (op.flags & kRunRows) ? ot : 0u;
        d.t0 = gather_at(op.ttab, ot);
        d.t1 = gather_at(op.ttab + 1, ot);
        d.t2 = gather_at(op.ttab + 2, ot);
        fetch_emit(op, d);
    };
    float mx = 0.f, my = 0.f, mz = 1.f;  // M / M0
    auto emit = [&](const Meta &op, const Rows &d) {
        float er = d.ex.x, ei = d.ex.y;
        cmul(er, ei, d.ez.x, d.ez.y);
        cmul(er, ei, mx, my);
        if (!act) er = ei = 0.f;
#pragma unroll
        for (int p = 0; p < MC; ++p) {
            if (p >= n_coils) break;
            float sr = er, si = ei;
            cmul(sr, si, d.y[p].x, d.y[p].y);
            seg_add<0x111>(m1, sr);
            seg_add<0x111>(m1, si);
            seg_add<0x112>(m2, sr);
            seg_add<0x112>(m2, si);
            seg_add<0x114>(m4, sr);
            seg_add<0x114>(m4, si);
            seg_add<0x118>(m8, sr);
            seg_add<0x118>(m8, si);
            seg_add<0x142>(mb15, sr);
            seg_add<0x142>(mb15, si);
            seg_add<0x143>(mb31, sr);
            seg_add<0x143>(mb31, si);
            if (end) {
                double2 *g = op.gsum + (int64_t)(coil0 + p) * op.stride + gx;
                if (own) {
                    store_pair(g, (double)sr, (double)si);
                } else {
                    group_add(&g->x, (double)sr);
                    group_add(&g->y, (double)si);
                }
            }
        }
    };
    auto full = [&](const Meta &op, const Rows &d) {
        float fr = d.px.x, fi = d.px.y;
        cmul(fr, fi, d.pz.x, d.pz.y);
        cmul(mx, my, fr, fi);
        if (op.flags & kPreMz) mz = fmaf(d.px.z, mz - 1.f, 1.f);
        if (op.flags & kOpRf) {
            // (the diagonal term, the largest, last: one rounding of its size)
            const float px = fmaf(d.t0.y, my, fmaf(d.t0.z, mz, d.t0.w));
            const float py = fmaf(d.t1.x, mx, fmaf(d.t1.z, mz, d.t1.w));
            const float pz = fmaf(d.t2.x, mx, fmaf(d.t2.y, my, d.t2.w));
            mx = fmaf(d.t0.x, mx, px);
            my = fmaf(d.t1.y, my, py);
            mz = fmaf(d.t2.z, mz, pz);
        }
        if (op.flags & kOpEmit) emit(op, d);
    };
    // Rows d[k] belong to operation o + k: used, then filled again kDepth ahead
    // (a copy of a register that a load still fills would wait for it).
    auto walk = [&](auto depth, const RunPart &part, auto fetch, auto apply) {
        constexpr int kDepth = decltype(depth)::value;
        const RunOp *ops = a.ops + part.first;
        const int n = part.n;
        Meta meta[kDepth];
        Rows d[kDepth];
#pragma unroll
        for (int k = 0; k < kDepth; ++k) {
            const RunOp op = load_desc(ops, min(k, n - 1));
            meta[k] = Meta{op.flags, op.gsum_stride, op.gsum};
            fetch(op, d[k]);
        }
        int o = 0;
        for (; o + kDepth <= n; o += kDepth) {
#pragma unroll
            for (int k = 0; k < kDepth; ++k) {
                const RunOp op = load_desc(ops, min(o + k + kDepth, n - 1));
                apply(meta[k], d[k]);
                meta[k] = Meta{op.flags, op.gsum_stride, op.gsum};
                fetch(op, d[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < kDepth - 1; ++k)
            if (o + k < n) apply(meta[k], d[k]);
    };
    for (int q = 0; q < a.n_parts; ++q) {
        const RunPart part = a.parts[q];
        if (part.emit_only)
            walk(std::integral_constant<int, MC == 1 ? 8 : 4>{}, part, fetch_emit, emit);
        else
            walk(std::integral_constant<int, MC == 1 ? 4 : 2>{}, part, fetch_full, full);
    }
    if (act && coil0 == 0) a.m[a.slot[r]] = make_float4(mx, my, mz, 0.f);
}

hipError_t launch_run_sweep(const RunSweepArgs &a, hipStream_t st) {
    if (a.n_waves <= 0) return hipSuccess;
    if (a.n_parts < 1 || a.n_parts > kRunMaxParts || a.n_coils < 1 || a.n_coils > 8 || a.r0 % kRunTile) return hipErrorInvalidValue;
    if (a.n_runs > kRunMaxRuns || a.n_lines > (1 << 20)) return hipErrorInvalidValue;  // 32-bit byte offsets
    // Several coils: four per wavefront, which repeats the steps of its runs for
    // each four.  With all eight in one the chip had a wavefront per SIMD or
    // less.  EPI of 128 lines with 8 coils, us per call: 29 k isochromats 267 and
    // 208, 595 k 443 and 381; 6.8 M (256 lines) 3084 and 3083, the kernel itself
    // 934 and 872 (two coils per wavefront 1012, one 1320).
    if (a.n_coils == 1)
        hipLaunchKernelGGL(k_run_sweep<1>, dim3((unsigned)a.n_waves), dim3(64), 0, st, a);
    else
        hipLaunchKernelGGL(k_run_sweep<4>, dim3((unsigned)a.n_waves, (unsigned)((a.n_coils + 3) / 4)), dim3(64), 0, st, a);
    return hipGetLastError();
}

// ------------------------------------------------------------- k_run_state
// One read of M0, the run index and the run's ratio (16 bytes, in L2) and one
// write of M per isochromat: 20 bytes of memory traffic.  V = 4: four
// isochromats per thread with 16-byte accesses.  The ratios lie in the order of
// the runs' first isochromats, so that neighbours of a grid row read
// neighbouring rows.
template <int V>
__global__ __launch_bounds__(256) void k_run_state(RunStateArgs a, int64_t n) {
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= n) return;
    int run[V];
    float m0[V], yv[V], o[3][V];
    if (V == 4) {
        ld4i((const int4 *)a.run, q, run);
        ld4((const float4 *)a.m0, q, m0);
        if (a.cy != 0.0) ld4((const float4 *)a.y, q, yv);
    } else {
        run[0] = a.run[q];
        m0[0] = a.m0[q];
        if (a.cy != 0.0) yv[0] = a.y[q];
    }
#pragma unroll
    for (int c = 0; c < V; ++c) {
        const float4 m = gather_row(a.m, run[c]);
        if (a.cy != 0.0) {  // in FP64, rounded once
            float s, co;
            sincos_rev(a.cy * (double)yv[c], &s, &co);
            // (turns of 0 and 1/2 are exact)
            const double w = (s == 0.f ? 1.0 : 1.0 + kTurnBias) * (double)m0[c], x = m.x, y = m.y;
            o[0][c] = (float)(w * (x * co + y * s));
            o[1][c] = (float)(w * (y * co - x * s));
        } else {
            o[0][c] = m.x * m0[c];
            o[1][c] = m.y * m0[c];
        }
        o[2][c] = m.z * m0[c];
    }
    float *out[3] = {a.ox, a.oy, a.oz};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        if (V == 4)
            ((float4 *)out[p])[q] = make_float4(o[p][0], o[p][1], o[p][2], o[p][3]);
        else
            out[p][q] = o[p][0];
    }
}

hipError_t launch_run_state(const RunStateArgs &a, hipStream_t st) {
    // ox, oy, oz are K floats apart
    const bool by4 = a.K % 4 == 0 && ((uintptr_t)a.ox | (uintptr_t)a.m0 | (uintptr_t)a.y | (uintptr_t)a.run) % 16 == 0;
    const int64_t n = by4 ? a.K / 4 : a.K, blocks = (n + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (by4)
        hipLaunchKernelGGL(k_run_state<4>, dim3((unsigned)blocks), dim3(256), 0, st, a, n);
    else
        hipLaunchKernelGGL(k_run_state<1>, dim3((unsigned)blocks), dim3(256), 0, st, a, n);
    return hipGetLastError();
}

}  // namespace gbs
