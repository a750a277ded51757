// Grouping of isochromats (Sec. 2.4, Fig. 2) on the device.
//
// For an axis a the key of isochromat k is (r_a, T1, T2, dB0), compared by
// exact bit pattern with -0 folded onto +0.  Keys are made order-preserving
// 32-bit words, packed as two 64-bit halves and sorted with two stable LSD
// radix passes (low half, then high half), carrying the isochromat index.
// Equal neighbours share a group id; ids are dense in lexicographic key order
// (z groups: of the key (T1, T2, dB0, z)).
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "groups.hpp"
#include "kernels.hpp"

namespace gbs {

// rocPRIM device primitives on int32 counts (stable LSD radix sort of 64-bit
// keys with an int32 payload; inclusive and exclusive sums).  With tmp null
// they report the temporary bytes they need in *bytes.
static hipError_t sort_pairs(void *tmp, size_t *bytes, const uint64_t *kin, uint64_t *kout, const int32_t *vin,
                             int32_t *vout, int64_t n, hipStream_t st) {
    return rocprim::radix_sort_pairs(tmp, *bytes, kin, kout, vin, vout, (unsigned int)n, 0u, 64u, st);
}
static hipError_t inclusive_sum(void *tmp, size_t *bytes, const int32_t *in, int32_t *out, int64_t n, hipStream_t st) {
    return rocprim::inclusive_scan(tmp, *bytes, in, out, (size_t)n, rocprim::plus<int32_t>(), st);
}
static hipError_t exclusive_sum(void *tmp, size_t *bytes, const int32_t *in, int32_t *out, int64_t n, hipStream_t st) {
    return rocprim::exclusive_scan(tmp, *bytes, in, out, (int32_t)0, (size_t)n, rocprim::plus<int32_t>(), st);
}

__device__ __forceinline__ uint32_t ordered_bits(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);  // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__global__ void k_keys(int64_t K, const float *__restrict__ a, const float *__restrict__ b,
                       const float *__restrict__ c, const float *__restrict__ d, uint64_t *hi,
                       uint64_t *lo, int32_t *idx) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        hi[i] = ((uint64_t)ordered_bits(a[i]) << 32) | ordered_bits(b[i]);
        lo[i] = ((uint64_t)ordered_bits(c[i]) << 32) | ordered_bits(d[i]);
        idx[i] = (int32_t)i;
    }
}

__global__ void k_gather_u64(int64_t K, const uint64_t *__restrict__ src, const int32_t *__restrict__ idx,
                             uint64_t *__restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[idx[i]];
}

__global__ void k_heads(int64_t K, const uint64_t *__restrict__ hi, const uint64_t *__restrict__ lo,
                        int32_t *__restrict__ flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x)
        flag[i] = (i == 0 || hi[i] != hi[i - 1] || lo[i] != lo[i - 1]) ? 1 : 0;
}

// ids = inclusive scan of the head flags (1-based).
__global__ void k_assign(int64_t K, const int32_t *__restrict__ ids, const int32_t *__restrict__ order,
                         const float *__restrict__ c, const float *__restrict__ t1,
                         const float *__restrict__ t2, const float *__restrict__ df,
                         int32_t *__restrict__ gid_nat, float4 *__restrict__ gtab,
                         int32_t *__restrict__ gstart) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = ids[i] - 1;
        const int32_t k = order[i];
        gid_nat[k] = g;
        if (i == 0 || ids[i - 1] != ids[i]) {
            gtab[g] = make_float4(c[k], t1[k], t2[k], df[k]);
            gstart[g] = (int32_t)i;
        }
    }
}

__global__ void k_counts(int64_t G, int64_t K, const int32_t *__restrict__ gstart, int32_t *__restrict__ gcount) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < G; g += (int64_t)gridDim.x * blockDim.x)
        gcount[g] = (int32_t)((g + 1 < G ? gstart[g + 1] : K) - gstart[g]);
}

__global__ void k_gather_f32(int64_t K, int64_t Kpad, const int32_t *__restrict__ perm,
                             const float *__restrict__ src, float *__restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < Kpad; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = i < K ? src[perm[i]] : 0.0f;
}

__global__ void k_gather_i32(int64_t K, int64_t Kpad, const int32_t *__restrict__ perm,
                             const int32_t *__restrict__ src, int32_t *__restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < Kpad; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = i < K ? src[perm[i]] : 0;
}

__global__ void k_validate(int64_t K, PhantomPtrs ph, int *bad) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        const float t1 = ph.t1[i], t2 = ph.t2[i];
        const bool ok = (t1 > 0.f) && (t2 > 0.f) && isfinite(ph.x[i]) && isfinite(ph.y[i]) &&
                        isfinite(ph.z[i]) && isfinite(ph.df[i]) && isfinite(ph.m0[i]);
        if (!ok) atomicOr(bad, 1);
    }
}

// ---- padded group-sorted layout ---------------------------------------------
// Isochromats are ordered by (x-group, z-group, index) and every run of equal
// (x-group, z-group) is padded to a multiple of 8 with copies of its first
// member carrying M0 = 0.  A thread's 8 (or 4) consecutive isochromats then always
// share both groups.
__global__ void k_pair_keys(int64_t K, const int32_t *__restrict__ gx, const int32_t *__restrict__ gz,
                            uint64_t *__restrict__ key, int32_t *__restrict__ idx) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        key[i] = ((uint64_t)(uint32_t)gx[i] << 32) | (gz ? (uint32_t)gz[i] : 0u);
        idx[i] = (int32_t)i;
    }
}

__global__ void k_key_heads(int64_t K, const uint64_t *__restrict__ key, int32_t *__restrict__ flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x)
        flag[i] = (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}

__global__ void k_run_start(int64_t K, const int32_t *__restrict__ rid, int32_t *__restrict__ rstart) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x)
        if (i == 0 || rid[i] != rid[i - 1]) rstart[rid[i] - 1] = (int32_t)i;
}

__global__ void k_run_plen(int64_t R, int64_t K, const int32_t *__restrict__ rstart, int32_t *__restrict__ plen) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t L = (int32_t)((r + 1 < R ? rstart[r + 1] : K) - rstart[r]);
        plen[r] = (L + 7) & ~7;  // 8-isochromat sweep threads never straddle a run
    }
}

__global__ void k_place(int64_t K, const int32_t *__restrict__ rid, const int32_t *__restrict__ rstart,
                        const int32_t *__restrict__ pstart, const int32_t *__restrict__ order,
                        int32_t *__restrict__ perm, int32_t *__restrict__ src) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = rid[i] - 1;
        const int64_t pos = (int64_t)pstart[r] + (i - rstart[r]);
        perm[pos] = order[i];
        src[pos] = order[i];
    }
}

__global__ void k_pad(int64_t R, int64_t K, const int32_t *__restrict__ rstart, const int32_t *__restrict__ pstart,
                      const int32_t *__restrict__ plen, const int32_t *__restrict__ order, int32_t *__restrict__ perm,
                      int32_t *__restrict__ src) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t L = (int32_t)((r + 1 < R ? rstart[r + 1] : K) - rstart[r]);
        const int32_t first = order[rstart[r]];
        for (int32_t j = L; j < plen[r]; ++j) {
            perm[pstart[r] + j] = -1;
            src[pstart[r] + j] = first;
        }
    }
}

__global__ void k_fill_tail(int64_t from, int64_t to, int32_t *__restrict__ perm, int32_t *__restrict__ src) {
    for (int64_t i = from + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < to; i += (int64_t)gridDim.x * blockDim.x) {
        perm[i] = -1;
        src[i] = 0;
    }
}

__global__ void k_zero_padding(int64_t n, const int32_t *__restrict__ perm, float *__restrict__ m0) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (perm[i] < 0) m0[i] = 0.0f;
}

static dim3 grid_for(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return dim3((unsigned)g);
}

hipError_t launch_validate_phantom(int64_t K, const PhantomPtrs &ph, int *bad, hipStream_t st) {
    hipLaunchKernelGGL(k_validate, grid_for(K), dim3(256), 0, st, K, ph, bad);
    return hipGetLastError();
}

hipError_t launch_gather_f32(int64_t K, int64_t Kpad, const int32_t *perm, const float *src, float *dst,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_gather_f32, grid_for(Kpad), dim3(256), 0, st, K, Kpad, perm, src, dst);
    return hipGetLastError();
}

hipError_t launch_gather_i32(int64_t K, int64_t Kpad, const int32_t *perm, const int32_t *src,
                             int32_t *dst, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_i32, grid_for(Kpad), dim3(256), 0, st, K, Kpad, perm, src, dst);
    return hipGetLastError();
}

__global__ void k_gather_padded(int64_t n, const int32_t *__restrict__ perm, const float *__restrict__ src,
                                float *__restrict__ dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t k = perm[i];
        dst[i] = k >= 0 ? src[k] : 0.0f;
    }
}

__global__ void k_check_finite(int64_t n, const float *__restrict__ a, int *__restrict__ bad) {
    bool ok = true;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        ok = ok && isfinite(a[i]);
    if (!ok) *bad = 1;
}

__global__ void k_expand_rows(const double *__restrict__ src, const int32_t *__restrict__ map, int64_t n,
                              double *__restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= 12 * n) return;
    const int64_t g = i / 12;
    dst[i] = src[12 * (int64_t)map[g] + (i - 12 * g)];
}

hipError_t launch_gather_padded(int64_t n, const int32_t *perm, const float *src, float *dst, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_padded, grid_for(n), dim3(256), 0, st, n, perm, src, dst);
    return hipGetLastError();
}

hipError_t launch_check_finite(int64_t n, const float *a, int *bad, hipStream_t st) {
    hipLaunchKernelGGL(k_check_finite, grid_for(n), dim3(256), 0, st, n, a, bad);
    return hipGetLastError();
}

hipError_t launch_expand_rows(const double *src, const int32_t *map, int64_t n, double *dst, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand_rows, dim3((unsigned)((12 * n + 255) / 256)), dim3(256), 0, st, src, map, n, dst);
    return hipGetLastError();
}

// Build the padded layout from natural-order x (and optional z) group ids.
// perm[pos] = isochromat at internal position pos or -1 (padding); src[pos] =
// the isochromat whose parameters the position copies.  perm/src need room
// for Kpad_cap entries; *kint receives the padded count (a multiple of 8).
hipError_t build_layout(int64_t K, const int32_t *gid_x, const int32_t *gid_z, void *scratch, size_t scratch_bytes,
                        int32_t *perm, int32_t *src, int64_t Kpad_cap, int64_t *kint, hipStream_t st) {
    char *p = (char *)scratch;
    auto take = [&](size_t n) {
        char *r = p;
        p += (n + 255) & ~(size_t)255;
        return (void *)r;
    };
    uint64_t *key = (uint64_t *)take(8 * K), *key2 = (uint64_t *)take(8 * K);
    int32_t *idx = (int32_t *)take(4 * K), *order = (int32_t *)take(4 * K), *flag = (int32_t *)take(4 * K);
    int32_t *rid = (int32_t *)take(4 * K), *rstart = (int32_t *)take(4 * K), *plen = (int32_t *)take(4 * K);
    int32_t *pstart = (int32_t *)take(4 * K);
    const size_t used = (size_t)(p - (char *)scratch);
    if (used > scratch_bytes) return hipErrorInvalidValue;
    void *tmp = p;
    size_t tmp_bytes = scratch_bytes - used;
    const dim3 g = grid_for(K);
    hipError_t e;
    hipLaunchKernelGGL(k_pair_keys, g, dim3(256), 0, st, K, gid_x, gid_z, key, idx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sort_pairs(tmp, &tmp_bytes, key, key2, idx, order, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_key_heads, g, dim3(256), 0, st, K, key2, flag);
    if ((e = inclusive_sum(tmp, &tmp_bytes, flag, rid, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_run_start, g, dim3(256), 0, st, K, rid, rstart);
    int32_t R = 0;
    if ((e = hipMemcpyAsync(&R, rid + (K - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_run_plen, grid_for(R), dim3(256), 0, st, (int64_t)R, K, rstart, plen);
    if ((e = exclusive_sum(tmp, &tmp_bytes, plen, pstart, R, st)) != hipSuccess) return e;
    int32_t last[2] = {0, 0};
    if ((e = hipMemcpyAsync(&last[0], pstart + (R - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipMemcpyAsync(&last[1], plen + (R - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    const int64_t n = (int64_t)last[0] + last[1];
    if (n > Kpad_cap) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_place, g, dim3(256), 0, st, K, rid, rstart, pstart, order, perm, src);
    hipLaunchKernelGGL(k_pad, grid_for(R), dim3(256), 0, st, (int64_t)R, K, rstart, pstart, plen, order, perm, src);
    if (Kpad_cap > n) hipLaunchKernelGGL(k_fill_tail, grid_for(Kpad_cap - n), dim3(256), 0, st, n, Kpad_cap, perm, src);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    *kint = n;
    return hipSuccess;
}

// ---- runs of the layout -------------------------------------------------------
__global__ void k_run_ids(int64_t n4, int32_t *__restrict__ ids, const int32_t *__restrict__ gid_x,
                          const int32_t *__restrict__ gid_z, int32_t *__restrict__ first4, int32_t *__restrict__ gx,
                          int32_t *__restrict__ gz) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n4; q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = ids[q];  // inclusive scan of the run starts, 1-based
        const int32_t x = gid_x[4 * q], z = gid_z[4 * q];
        if (q == 0 || x != gid_x[4 * q - 4] || z != gid_z[4 * q - 4]) {
            first4[r - 1] = (int32_t)q;
            gx[r - 1] = x;
            gz[r - 1] = z;
        }
        if (q == n4 - 1) first4[r] = (int32_t)n4;
    }
}

// xrun[g] <- first run of x-group g, xrun[G] <- the number of runs
__global__ void k_group_runs(int64_t n_runs, const int32_t *__restrict__ gx, int64_t n_groups,
                             int32_t *__restrict__ xrun) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= n_runs; r += (int64_t)gridDim.x * blockDim.x) {
        if (r == n_runs)
            xrun[n_groups] = (int32_t)n_runs;
        else if (r == 0 || gx[r - 1] != gx[r])
            xrun[gx[r]] = (int32_t)r;
    }
}

__global__ void k_run_starts(int64_t n4, const int32_t *__restrict__ gid_x, const int32_t *__restrict__ gid_z,
                             int32_t *__restrict__ flag) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n4; q += (int64_t)gridDim.x * blockDim.x)
        flag[q] = q == 0 || gid_x[4 * q] != gid_x[4 * q - 4] || gid_z[4 * q] != gid_z[4 * q - 4];
}

__global__ void k_first_flags(int64_t R, const int32_t *__restrict__ first4, const int32_t *__restrict__ perm,
                              int32_t *__restrict__ flag) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x)
        flag[perm[4 * (int64_t)first4[r]]] = 1;  // a run's first slot holds its first isochromat
}

__global__ void k_run_slots(int64_t R, const int32_t *__restrict__ first4, const int32_t *__restrict__ perm,
                            const int32_t *__restrict__ rank, int32_t *__restrict__ slot) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x)
        slot[r] = rank[perm[4 * (int64_t)first4[r]]];
}

__global__ void k_run_of(int64_t K, const int32_t *__restrict__ inv, const int32_t *__restrict__ run_of4,
                         const int32_t *__restrict__ slot, int32_t *__restrict__ run) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x)
        run[k] = slot[run_of4[inv[k] >> 2]];
}

__global__ void k_zero_i32(int64_t n, int32_t *v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v[i] = 0;
}

__global__ void k_minus_one(int64_t n, int32_t *v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v[i] -= 1;
}

// Numbers the runs of equal (x-group, z-group) of the layout's n4 quads in
// layout order: run_of4[q] (1-based until launch_run_arrays), and the count
// through *n_runs (synchronizes the stream).  scratch: room for n4 int32 and
// the scan's temporary memory.
hipError_t number_runs(int64_t n4, const int32_t *gid_x, const int32_t *gid_z, void *scratch, size_t scratch_bytes,
                       int32_t *run_of4, int64_t *n_runs, hipStream_t st) {
    int32_t *flag = (int32_t *)scratch;
    const size_t used = (4 * (size_t)n4 + 255) & ~(size_t)255;
    if (used > scratch_bytes) return hipErrorInvalidValue;
    size_t tmp_bytes = 0;
    hipError_t e = inclusive_sum(nullptr, &tmp_bytes, nullptr, nullptr, n4, st);
    if (e != hipSuccess) return e;
    if (used + tmp_bytes > scratch_bytes) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_run_starts, grid_for(n4), dim3(256), 0, st, n4, gid_x, gid_z, flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = inclusive_sum((char *)scratch + used, &tmp_bytes, flag, run_of4, n4, st)) != hipSuccess) return e;
    int32_t last = 0;
    if ((e = hipMemcpyAsync(&last, run_of4 + (n4 - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    *n_runs = last;
    return hipSuccess;
}

// slot[r]: rank of run r by its first isochromat in the caller's order; run[k]:
// slot of isochromat k's run.  run_of4 0-based.  scratch: 2 K int32 and the scan.
hipError_t place_runs(int64_t K, int64_t R, const int32_t *first4, const int32_t *run_of4, const int32_t *perm,
                      const int32_t *inv, void *scratch, size_t scratch_bytes, int32_t *slot, int32_t *run,
                      hipStream_t st) {
    const size_t one = (4 * (size_t)K + 255) & ~(size_t)255;
    int32_t *flag = (int32_t *)scratch, *rank = (int32_t *)((char *)scratch + one);
    size_t tmp_bytes = 0;
    hipError_t e = exclusive_sum(nullptr, &tmp_bytes, nullptr, nullptr, K, st);
    if (e != hipSuccess) return e;
    if (2 * one + tmp_bytes > scratch_bytes) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zero_i32, grid_for(K), dim3(256), 0, st, K, flag);
    hipLaunchKernelGGL(k_first_flags, grid_for(R), dim3(256), 0, st, R, first4, perm, flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = exclusive_sum((char *)scratch + 2 * one, &tmp_bytes, flag, rank, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_run_slots, grid_for(R), dim3(256), 0, st, R, first4, perm, rank, slot);
    hipLaunchKernelGGL(k_run_of, grid_for(K), dim3(256), 0, st, K, inv, run_of4, slot, run);
    return hipGetLastError();
}

// first4[r] (and n4 after the last run), x- and z-group of every run from the
// numbering of number_runs, whose run_of4 becomes 0-based.
hipError_t launch_run_arrays(int64_t n4, int32_t *run_of4, const int32_t *gid_x, const int32_t *gid_z,
                             int32_t *first4, int32_t *gx, int32_t *gz, hipStream_t st) {
    hipLaunchKernelGGL(k_run_ids, grid_for(n4), dim3(256), 0, st, n4, run_of4, gid_x, gid_z, first4, gx, gz);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_minus_one, grid_for(n4), dim3(256), 0, st, n4, run_of4);
    return hipGetLastError();
}

hipError_t launch_group_runs(int64_t n_runs, const int32_t *gx, int64_t n_groups, int32_t *xrun, hipStream_t st) {
    hipLaunchKernelGGL(k_group_runs, grid_for(n_runs + 1), dim3(256), 0, st, n_runs, gx, n_groups, xrun);
    return hipGetLastError();
}

__global__ void k_invert(int64_t n, const int32_t *__restrict__ perm, int32_t *__restrict__ inv) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (perm[i] >= 0) inv[perm[i]] = (int32_t)i;
}

hipError_t launch_invert(int64_t n, const int32_t *perm, int32_t *inv, hipStream_t st) {
    hipLaunchKernelGGL(k_invert, grid_for(n), dim3(256), 0, st, n, perm, inv);
    return hipGetLastError();
}

hipError_t launch_zero_padding(int64_t n, const int32_t *perm, float *m0, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_padding, grid_for(n), dim3(256), 0, st, n, perm, m0);
    return hipGetLastError();
}

size_t group_scratch_bytes(int64_t K) {
    size_t sort_tmp = 0, scan_tmp = 0, escan_tmp = 0;
    const bool sized = sort_pairs(nullptr, &sort_tmp, nullptr, nullptr, nullptr, nullptr, K, 0) == hipSuccess &&
                       inclusive_sum(nullptr, &scan_tmp, nullptr, nullptr, K, 0) == hipSuccess &&
                       exclusive_sum(nullptr, &escan_tmp, nullptr, nullptr, K, 0) == hipSuccess;
    size_t tmp = sort_tmp > scan_tmp ? sort_tmp : scan_tmp;
    if (escan_tmp > tmp) tmp = escan_tmp;
    // a failed size query leaves generous room; the sorts and scans report their own errors
    if (!sized) tmp = ((size_t)64 << 20) + 16 * (size_t)K;
    // the larger of group_axis (4 u64 + 3 i32 arrays) and build_layout (2 u64 + 7 i32), plus tmp
    return 4 * sizeof(uint64_t) * K + 7 * sizeof(int32_t) * K + tmp + 16 * 256;
}

// Group one axis, ids in the order of (coord, T1, T2, df) or, with coord_last,
// (T1, T2, df, coord): the z-groups of one tissue then are neighbours, and so
// are the transition rows that the runs of an x-group read (one tissue,
// successive z).  coord = r_a of every isochromat (natural order).  Writes
// gid_nat[K] (natural order), gtab[n_groups] = (coord, T1, T2, df) and
// gcount[n_groups] (gtab and gcount need room for K entries), order[K] =
// isochromat indices sorted by key (stable), and returns the group count
// through *n_groups (synchronizes the stream).
hipError_t group_axis(int64_t K, bool coord_last, const float *coord, const float *t1, const float *t2, const float *df,
                      void *scratch, size_t scratch_bytes, int32_t *gid_nat, float4 *gtab,
                      int32_t *gcount, int32_t *order, int64_t *n_groups, hipStream_t st) {
    char *p = (char *)scratch;
    auto take = [&](size_t n) {
        char *r = p;
        p += (n + 255) & ~(size_t)255;
        return (void *)r;
    };
    uint64_t *hi = (uint64_t *)take(8 * K), *lo = (uint64_t *)take(8 * K);
    uint64_t *k2 = (uint64_t *)take(8 * K), *k3 = (uint64_t *)take(8 * K);
    int32_t *idx0 = (int32_t *)take(4 * K), *idx1 = (int32_t *)take(4 * K), *flag = (int32_t *)take(4 * K);
    const size_t used = (size_t)(p - (char *)scratch);
    if (used > scratch_bytes) return hipErrorInvalidValue;
    void *tmp = p;
    size_t tmp_bytes = scratch_bytes - used;
    const dim3 g = grid_for(K);
    hipError_t e;
    if (coord_last)
        hipLaunchKernelGGL(k_keys, g, dim3(256), 0, st, K, t1, t2, df, coord, hi, lo, idx0);
    else
        hipLaunchKernelGGL(k_keys, g, dim3(256), 0, st, K, coord, t1, t2, df, hi, lo, idx0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // LSD: low half first (carry indices), then the high half of the same records.
    if ((e = sort_pairs(tmp, &tmp_bytes, lo, k2, idx0, idx1, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_gather_u64, g, dim3(256), 0, st, K, hi, idx1, k3);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sort_pairs(tmp, &tmp_bytes, k3, hi, idx1, order, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_gather_u64, g, dim3(256), 0, st, K, lo, order, k2);  // low half in final order
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_heads, g, dim3(256), 0, st, K, hi, k2, flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = inclusive_sum(tmp, &tmp_bytes, flag, idx0, K, st)) != hipSuccess) return e;
    int32_t *gstart = idx1;  // the first sort's payload is no longer needed
    hipLaunchKernelGGL(k_assign, g, dim3(256), 0, st, K, idx0, order, coord, t1, t2, df, gid_nat, gtab, gstart);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int32_t last = 0;
    if ((e = hipMemcpyAsync(&last, idx0 + (K - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_counts, grid_for(last), dim3(256), 0, st, (int64_t)last, K, gstart, gcount);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    *n_groups = last;
    return hipSuccess;
}

}  // namespace gbs
