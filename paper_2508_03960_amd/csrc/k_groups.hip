// Grouping of isochromats (Sec. 2.4, Fig. 2) on the device.
//
// For an axis a the key of isochromat k is (r_a, T1, T2, dB0), compared by
// exact bit pattern with -0 folded onto +0.  Equal keys share a group id; ids
// are dense in lexicographic key order (z groups: of the key (T1, T2, dB0, z)).
//
// Two ways to the same ids:
//  dense (dense_fields, dense_groups): the distinct values of every field are
//      found and ranked; a key is then a cell of the product of the fields,
//      and the ids are a scan over the occupied cells.  Three passes over the
//      isochromats for all axes together, without a sort: 0.35 ms for 6.8 M
//      isochromats on a 512 x 512 x 26 grid with 6 T1, 6 T2 and 16 dB0.
//  sorted (group_axis): the key packed as two 64-bit halves, sorted with two
//      stable LSD radix passes (low half, then high half), carrying the
//      isochromat index: 1.3 ms for each of the three axes of that phantom.
// A phantom takes the dense way while no field has more than kFieldCap
// distinct values and all axes together at most dense_cell_limit cells, which
// bounds the scan by one more pass over the isochromats; arbitrary positions
// or a measured dB0 map are sorted.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include "groups.hpp"
#include "kernels.hpp"

namespace gbs {

// rocPRIM device primitives on int32 counts (stable LSD radix sort of the low
// `bits` bits of 64-bit keys with an int32 payload; inclusive and exclusive
// sums).  One key type for all sorts: a second one doubles the code to load for
// a tenth of a pass.  With tmp null they report the temporary bytes they need in
// *bytes.
static hipError_t sort_pairs(void *tmp, size_t *bytes, const uint64_t *kin, uint64_t *kout, const int32_t *vin,
                             int32_t *vout, int64_t n, unsigned int bits, hipStream_t st) {
    return rocprim::radix_sort_pairs(tmp, *bytes, kin, kout, vin, vout, (unsigned int)n, 0u, bits, st);
}
template <typename In>
static hipError_t inclusive_sum(void *tmp, size_t *bytes, In in, int32_t *out, int64_t n, hipStream_t st) {
    return rocprim::inclusive_scan(tmp, *bytes, in, out, (size_t)n, rocprim::plus<int32_t>(), st);
}
static hipError_t exclusive_sum(void *tmp, size_t *bytes, const int32_t *in, int32_t *out, int64_t n, hipStream_t st) {
    return rocprim::exclusive_scan(tmp, *bytes, in, out, (int32_t)0, (size_t)n, rocprim::plus<int32_t>(), st);
}

// 1 where a run of the sorted keys starts: where a key differs from the one
// before it, and inside longer stretches of one key at the multiples of
// kRunPiece that have kRunPiece positions of it on either side.  So no run is
// longer than 3 kRunPiece - 2 positions, and a stretch below 2 kRunPiece is one
// run: a run's sum over its members (k_run_y) is one wavefront's work, and one
// run of 2^20 isochromats kept the whole chip waiting for 15.7 ms.
struct HeadFlag {
    const uint64_t *key;
    int64_t n;
    __device__ bool key_starts(int64_t i) const { return i == 0 || key[i] != key[i - 1]; }
    __device__ int32_t operator()(int64_t i) const {
        if (key_starts(i)) return 1;
        return i % kRunPiece == 0 && i + kRunPiece <= n && key[i - kRunPiece] == key[i + kRunPiece - 1];
    }
};
static auto head_flags(const uint64_t *key, int64_t n) {
    return rocprim::make_transform_iterator(rocprim::make_counting_iterator<int64_t>(0), HeadFlag{key, n});
}

__device__ __forceinline__ uint32_t ordered_bits(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);  // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t v) {
    return __uint_as_float((v & 0x80000000u) ? (v ^ 0x80000000u) : ~v);
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
                         int32_t *__restrict__ gid_nat) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x)
        gid_nat[order[i]] = ids[i] - 1;
}

__global__ void k_group_table(int64_t K, const int32_t *__restrict__ ids, const int32_t *__restrict__ order,
                              const float *__restrict__ c, const float *__restrict__ t1, const float *__restrict__ t2,
                              const float *__restrict__ df, float4 *__restrict__ gtab) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        if (i > 0 && ids[i - 1] == ids[i]) continue;
        const int32_t k = order[i];
        gtab[ids[i] - 1] = make_float4(c[k], t1[k], t2[k], df[k]);
    }
}

__global__ void k_validate(int64_t K, PhantomPtrs ph, int *bad) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        const float t1 = ph.t1[i], t2 = ph.t2[i];
        const bool ok = (t1 > 0.f) && (t2 > 0.f) && isfinite(ph.x[i]) && isfinite(ph.y[i]) &&
                        isfinite(ph.z[i]) && isfinite(ph.df[i]) && isfinite(ph.m0[i]);
        if (!ok) atomicOr(bad, 1);
    }
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

// ---- fields with few distinct values --------------------------------------------
// The distinct values of the key fields, each collected in a hash table of
// twice kFieldCap slots.  A workgroup keeps the values it has met in a table
// of its own in LDS, so that the shared one, whose probes must see the other
// dies' insertions and bypass the L2, sees each value once per workgroup (a
// direct-mapped LDS filter, which values of one slot evict from each other in
// turn, left 1.2 ms of such probes for 6.8 M isochromats).
// A value's ordered bits are never 0 (that pattern is a NaN, which no phantom
// holds): 0 marks an empty slot.  A workgroup that inserts a value beyond
// kFieldCap stops, and the field counts as given up; so does one whose probe
// finds many slots taken and the count beyond kFieldCap.  All probe loops end
// after one turn of their table at most.
constexpr int kSeen = 4096, kSeenProbes = 8, kValueBlocks = 512, kValueUnroll = 4;

__device__ __forceinline__ uint32_t hash_of(uint32_t v) { return v * 2654435761u; }

// v's place in the workgroup's table: true if it was there already
__device__ __forceinline__ bool seen_before(uint32_t *seen, uint32_t v) {
    uint32_t s = hash_of(v) >> 20;
    static_assert(kSeen == 1 << 12, "slot of a hash");
    for (int p = 0; p < kSeenProbes; ++p, s = (s + 1) % kSeen) {
        uint32_t cur = __hip_atomic_load(seen + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == 0) cur = atomicCAS(seen + s, 0u, v);
        if (cur == v) return true;
        if (cur == 0) return false;
    }
    return false;  // no room: v goes to the shared table each time
}

// Clears the tables; and gives up at once (count beyond kFieldCap) a field
// that has more than f.cap values among kSampled isochromats.  Where every
// isochromat has a value of its own (a measured dB0 map, free positions), the
// table below fills up under all of the chip's threads at once, and their probes
// past the L2 took 5 ms; this takes 15 us, beside the clearing.  Fields that
// pass have seldom more values than twice kFieldCap slots.
constexpr int kSampled = 3 * kFieldCap / 2, kSampleWG = 1024;

__global__ __launch_bounds__(kSampleWG) void k_field_start(int64_t K, Fields f, int64_t n_zero, int32_t *zero) {
    if (blockIdx.x >= kFields) {
        const int64_t stride = (int64_t)(gridDim.x - kFields) * kSampleWG;
        for (int64_t i = (int64_t)(blockIdx.x - kFields) * kSampleWG + threadIdx.x; i < n_zero; i += stride) zero[i] = 0;
        return;
    }
    __shared__ uint32_t seen[kFieldSlots];
    __shared__ int found;
    const float *val = f.val[blockIdx.x];
    if (!val || K <= f.cap) {
        if (threadIdx.x == 0) f.count[blockIdx.x] = 0;
        return;
    }
    for (int i = threadIdx.x; i < kFieldSlots; i += kSampleWG) seen[i] = 0;
    if (threadIdx.x == 0) found = 0;
    constexpr int kEach = kSampled / kSampleWG;
    const int n = K < kSampled ? (int)K : kSampled;
    uint32_t v[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int i = j * kSampleWG + threadIdx.x;
        v[j] = i < n ? ordered_bits(val[(int64_t)i * K / n]) : 0u;
    }
    __syncthreads();
    int mine = 0;
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        if (v[j] == 0) continue;
        uint32_t s = hash_of(v[j]) >> 18, cur;
        while ((cur = atomicCAS(seen + s, 0u, v[j])) != 0 && cur != v[j]) s = (s + 1) % kFieldSlots;  // (a quarter stays empty)
        mine += cur == 0;
    }
    atomicAdd(&found, mine);
    __syncthreads();
    if (threadIdx.x == 0) f.count[blockIdx.x] = found > f.cap ? kFieldCap + 1 : 0;
}

__global__ __launch_bounds__(256) void k_field_values(int64_t K, Fields f) {
    __shared__ uint32_t seen[kSeen];
    __shared__ int stop;
    const int q = blockIdx.y;
    const float *val = f.val[q];
    bool given_up = false;
    for (int p = 0; p < kFields; ++p) given_up = given_up || f.count[p] > f.cap;
    if (!val || given_up) return;
    for (int i = threadIdx.x; i < kSeen; i += 256) seen[i] = 0;
    if (threadIdx.x == 0) stop = 0;
    __syncthreads();
    uint32_t *set = f.set[q];
    int32_t *count = f.count + q;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < K; i0 += kValueUnroll * stride) {
        float x[kValueUnroll];
#pragma unroll
        for (int u = 0; u < kValueUnroll; ++u) x[u] = val[i0 + u * stride < K ? i0 + u * stride : i0];
#pragma unroll
        for (int u = 0; u < kValueUnroll; ++u) {
            const uint32_t v = ordered_bits(x[u]);
            if (v == 0 || seen_before(seen, v)) continue;
            uint32_t s = hash_of(v) >> 18;
            static_assert(kFieldSlots == 1 << 14, "slot of a hash");
            for (int probe = 1; probe <= kFieldSlots; ++probe, s = (s + 1) % kFieldSlots) {
                uint32_t cur = __hip_atomic_load(set + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (cur == 0) {
                    cur = atomicCAS(set + s, 0u, v);
                    if (cur == 0) {
                        const int32_t n = atomicAdd(count, 1);
                        if (n < kFieldCap)
                            f.list[q][n] = v;
                        else
                            stop = 1;
                        break;
                    }
                }
                if (cur == v) break;
                if (probe % 16 == 0 &&
                    __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > kFieldCap) {
                    stop = 1;
                    break;
                }
            }
        }
        if (__hip_atomic_load(&stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return;
    }
}

// A field's rank table has the smallest power of two of slots that leaves half
// of them empty, so that the lookups of a few hundred values stay in L1; a
// value's slot is the top bits of its hash, behind this shift.
__host__ __device__ __forceinline__ int rank_shift(int32_t count) {
    int s = 26;
    while (((uint32_t)1 << (32 - s)) < 2 * (uint32_t)count) --s;
    return s;
}

// rank of a value = number of smaller ones (at most kFieldCap compares, from LDS)
__global__ __launch_bounds__(256) void k_field_ranks(Fields f) {
    __shared__ uint32_t part[1024];
    const int q = blockIdx.y;
    const int32_t n = f.count[q];
    if (n > kFieldCap || (int64_t)blockIdx.x * 256 >= n) return;  // uniform
    const int i = blockIdx.x * 256 + threadIdx.x;
    const uint32_t v = i < n ? f.list[q][i] : 0u;
    int32_t r = 0;
    for (int c = 0; c < n; c += 1024) {
        __syncthreads();
        for (int j = threadIdx.x; j < 1024; j += 256) part[j] = c + j < n ? f.list[q][c + j] : 0xffffffffu;
        __syncthreads();
        for (int j = 0; j < 1024; ++j) r += part[j] < v;
    }
    if (i >= n) return;
    f.sorted[q][r] = v;
    const int sh = rank_shift(n);
    const uint32_t mask = (1u << (32 - sh)) - 1;
    const unsigned long long e = ((unsigned long long)v << 32) | (uint32_t)r;
    for (uint32_t s = hash_of(v) >> sh;; s = (s + 1) & mask)  // n <= half of the slots: ends at an empty one
        if (atomicCAS((unsigned long long *)f.rank[q] + s, 0ull, e) == 0ull) break;
}

__device__ __forceinline__ int32_t rank_of(const uint64_t *tab, int sh, float val) {
    const uint32_t v = ordered_bits(val), mask = (1u << (32 - sh)) - 1;
    uint32_t s = hash_of(v) >> sh;
    uint64_t e = tab[s];
    while ((uint32_t)(e >> 32) != v && e != 0) {  // every value is in its table
        s = (s + 1) & mask;
        e = tab[s];
    }
    return (int32_t)(uint32_t)e;
}

// base[0 .. 4] of the fields' counts; false if there are more than limit cells
static bool cell_blocks(const int32_t *count, int64_t limit, Cells &c) {
    int64_t nt = 1;
    for (int q = 3; q < kFields; ++q) {
        if (count[q] > kFieldCap || count[q] <= 0) return false;
        nt *= count[q];
        if (nt > limit) return false;
    }
    c.n2 = count[4];
    c.nd = count[5];
    c.nt = (int32_t)nt;
    c.base[0] = 0;
    for (int a = 0; a < 3; ++a) {
        if (count[a] > kFieldCap) return false;
        c.nc[a] = count[a];
        c.base[a + 1] = c.base[a] + (int64_t)count[a] * nt;
    }
    c.base[4] = c.base[3] + nt;
    for (int q = 0; q < kFields; ++q) c.shift[q] = rank_shift(count[q]);
    return c.base[4] <= limit;
}

// (an occupied cell's flag is written by whoever still reads 0: the same value)
__device__ __forceinline__ void mark(int32_t *flag, int64_t c) {
    if (flag[c] == 0) flag[c] = 1;
}

__global__ __launch_bounds__(256) void k_cells(int64_t K, Fields f, Cells c) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < K; i += (int64_t)gridDim.x * 256) {
        int32_t r[kFields];
#pragma unroll
        for (int q = 0; q < kFields; ++q) r[q] = f.val[q] ? rank_of(f.rank[q], c.shift[q], f.val[q][i]) : 0;
        const int32_t t = (r[3] * c.n2 + r[4]) * c.nd + r[5];
        mark(c.flag, c.base[3] + t);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (!f.val[a]) continue;
            const int32_t cell = a == 2 ? t * c.nc[a] + r[a] : r[a] * c.nt + t;
            c.gid[a][i] = cell;
            mark(c.flag, c.base[a] + cell);
        }
    }
}

// total[a] <- groups up to and with block a (a = 3: with the tissues)
__global__ void k_cell_totals(Cells c, int32_t *__restrict__ total) {
    const int a = threadIdx.x;
    if (a < 4) total[a] = c.base[a + 1] > 0 ? c.ids[c.base[a + 1] - 1] : 0;
}

__global__ __launch_bounds__(256) void k_cell_tables(Fields f, Cells c, const int32_t *__restrict__ total,
                                                     float4 *gtab0, float4 *gtab1, float4 *gtab2, float4 *ttab,
                                                     int32_t *tmap) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= c.base[4] || !c.flag[i]) return;
    const int a = i < c.base[1] ? 0 : i < c.base[2] ? 1 : i < c.base[3] ? 2 : 3;
    const int32_t cell = (int32_t)(i - c.base[a]);
    const int32_t t = a == 3 ? cell : a == 2 ? cell / c.nc[2] : cell % c.nt;
    const int32_t g = c.ids[i] - 1 - (a ? total[a - 1] : 0);
    float4 v = make_float4(0.f, from_ordered(f.sorted[3][t / (c.n2 * c.nd)]), from_ordered(f.sorted[4][t / c.nd % c.n2]),
                           from_ordered(f.sorted[5][t % c.nd]));
    if (a == 3) {
        if (ttab) ttab[g] = v;
        return;
    }
    v.x = from_ordered(f.sorted[a][a == 2 ? cell % c.nc[2] : cell / c.nt]);
    (a == 0 ? gtab0 : a == 1 ? gtab1 : gtab2)[g] = v;
    if (a == 0 && tmap) tmap[g] = c.ids[c.base[3] + t] - 1 - total[2];
}

// cell -> group, in place
__global__ __launch_bounds__(256) void k_cell_groups(int64_t K, Cells c, const int32_t *__restrict__ total) {
    const int32_t t0 = total[0], t1 = total[1];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < K; i += (int64_t)gridDim.x * 256) {
        if (c.nc[0]) c.gid[0][i] = c.ids[c.base[0] + c.gid[0][i]] - 1;
        if (c.nc[1]) c.gid[1][i] = c.ids[c.base[1] + c.gid[1][i]] - 1 - t0;
        if (c.nc[2]) c.gid[2][i] = c.ids[c.base[2] + c.gid[2][i]] - 1 - t1;
    }
}

__global__ void k_zero_i32(int64_t n, int32_t *v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v[i] = 0;
}

int64_t dense_cell_limit(int64_t K) { return K > (1 << 20) ? K : (1 << 20); }

constexpr size_t kFieldCounts = 64, kFieldTables = kFields * 3 * kFieldSlots;  // rank and value tables: zero at the start
constexpr size_t kFieldFound = kFields * 2 * kFieldCap;          // lists and sorted values

static bool carve_fields(const float *const val[kFields], int64_t cap, Carve &w, Fields &f) {
    int32_t *z = w.take<int32_t>(kFieldCounts + kFieldTables), *u = w.take<int32_t>(kFieldFound);
    if (!z || !u) return false;
    f.count = z;
    f.cap = (int32_t)(cap < kFieldCap ? cap : kFieldCap);
    for (int q = 0; q < kFields; ++q) {
        f.val[q] = val[q];
        f.rank[q] = (uint64_t *)(z + kFieldCounts) + q * kFieldSlots;
        f.set[q] = (uint32_t *)(z + kFieldCounts + kFields * 2 * kFieldSlots) + q * kFieldSlots;
        f.list[q] = (uint32_t *)u + q * 2 * kFieldCap;
        f.sorted[q] = f.list[q] + kFieldCap;
    }
    return true;
}

// The fields' distinct values; their counts to count[kFields] (asynchronous).
static hipError_t count_fields(int64_t K, const Fields &f, int32_t *count, hipStream_t st) {
    hipLaunchKernelGGL(k_field_start, dim3(kFields + (kFieldTables + kSampleWG - 1) / kSampleWG), dim3(kSampleWG), 0, st, K, f,
                       (int64_t)kFieldTables, f.count + kFieldCounts);
    const int64_t need = (K + 255) / 256;
    hipLaunchKernelGGL(k_field_values, dim3((unsigned)(need < kValueBlocks ? need : kValueBlocks), kFields), dim3(256), 0,
                       st, K, f);
    hipError_t e;
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipMemcpyAsync(count, f.count, sizeof(int32_t) * kFields, hipMemcpyDeviceToHost, st);
}

// Their rank tables, once the counts say that the phantom takes them.
static hipError_t rank_fields(const Fields &f, const int32_t *count, hipStream_t st) {
    int32_t most = 1;
    for (int q = 0; q < kFields; ++q) most = count[q] > most ? count[q] : most;
    hipLaunchKernelGGL(k_field_ranks, dim3((unsigned)((most + 255) / 256), kFields), dim3(256), 0, st, f);
    return hipGetLastError();
}

// Groups of all requested axes (coord[a] null: not requested) by cells; gid[a]
// has room for K.  *done stays false if the phantom needs the sorted way.
// Otherwise gid[a] holds the groups (natural order), d->total the group counts
// (synchronizes the stream), and dense_tables writes the tables while the
// scratch holds.
hipError_t dense_groups(int64_t K, const float *const coord[3], const float *t1, const float *t2, const float *df,
                        void *scratch, size_t scratch_bytes, int32_t *const gid[3], DenseGroups *d, bool *done,
                        hipStream_t st) {
    *done = false;
    Carve w{(char *)scratch, scratch_bytes};
    Fields &f = d->f;
    Cells &c = d->c;
    const float *const val[kFields] = {coord[0], coord[1], coord[2], t1, t2, df};
    if (!carve_fields(val, kFieldCap, w, f)) return hipErrorInvalidValue;
    int32_t count[kFields];
    hipError_t e = count_fields(K, f, count, st);
    if (e != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    if (!cell_blocks(count, dense_cell_limit(K), c)) return hipSuccess;
    if ((e = rank_fields(f, count, st)) != hipSuccess) return e;
    const int64_t n = c.base[4];
    d->d_total = w.take<int32_t>(4);
    c.flag = w.take<int32_t>((size_t)n);
    c.ids = w.take<int32_t>((size_t)n);
    size_t tmp_bytes = 0;
    if ((e = inclusive_sum(nullptr, &tmp_bytes, (const int32_t *)nullptr, nullptr, n, st)) != hipSuccess) return e;
    char *tmp = w.take<char>(tmp_bytes);
    if (!d->d_total || !c.flag || !c.ids || !tmp) return hipErrorInvalidValue;
    for (int a = 0; a < 3; ++a) c.gid[a] = gid[a];
    hipLaunchKernelGGL(k_zero_i32, grid_for(n), dim3(256), 0, st, n, c.flag);
    hipLaunchKernelGGL(k_cells, grid_for(K), dim3(256), 0, st, K, f, c);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = inclusive_sum(tmp, &tmp_bytes, (const int32_t *)c.flag, c.ids, n, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_cell_totals, dim3(1), dim3(64), 0, st, c, d->d_total);
    hipLaunchKernelGGL(k_cell_groups, grid_for(K), dim3(256), 0, st, K, c, (const int32_t *)d->d_total);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(d->total, d->d_total, sizeof(d->total), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    *done = true;
    return hipSuccess;
}

// gtab[a][group] = (coord, T1, T2, df) of every requested axis, and (or null)
// the tissues' (0, T1, T2, df) and the tissue of each x-group.
hipError_t dense_tables(const DenseGroups &d, float4 *const gtab[3], float4 *ttab, int32_t *tmap, hipStream_t st) {
    hipLaunchKernelGGL(k_cell_tables, dim3((unsigned)((d.c.base[4] + 255) / 256)), dim3(256), 0, st, d.f, d.c,
                       (const int32_t *)d.d_total, gtab[0], gtab[1], gtab[2], ttab, tmap);
    return hipGetLastError();
}

// ---- groups of the adjoint ------------------------------------------------------
// cell = (((x ny + y) nz + z) nd + dB0) C + class, of the values' ranks
struct AdjCells {
    int64_t n;
    int32_t nv[4], C;  // values of x, y, z (1: not compared), dB0; classes
    int32_t shift[4];
    int32_t *flag, *ids;
};

__device__ __forceinline__ int64_t adj_cell(const Fields &f, const AdjCells &c, const int32_t *cls, int64_t i) {
    int64_t cell = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (f.val[q]) cell = cell * c.nv[q] + rank_of(f.rank[q], c.shift[q], f.val[q][i]);
    return cell * c.C + cls[i];
}

__global__ __launch_bounds__(256) void k_adj_cells(int64_t K, Fields f, AdjCells c, const int32_t *__restrict__ cls,
                                                   uint64_t *__restrict__ cell) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < K; i += (int64_t)gridDim.x * 256) {
        const int64_t v = adj_cell(f, c, cls, i);
        cell[i] = (uint64_t)v;
        mark(c.flag, v);
    }
}

__global__ __launch_bounds__(256) void k_adj_tables(Fields f, AdjCells c, float4 *__restrict__ gtab,
                                                    int32_t *__restrict__ gcls) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= c.n || !c.flag[i]) return;
    const int32_t g = c.ids[i] - 1;
    int64_t r = i / c.C;
    float v[4];
#pragma unroll
    for (int q = 3; q >= 0; --q) {
        v[q] = f.val[q] ? from_ordered(f.sorted[q][r % c.nv[q]]) : 0.f;
        r /= c.nv[q];
    }
    gtab[g] = make_float4(v[0], v[1], v[2], v[3]);
    gcls[g] = (int32_t)(i % c.C);
}

__global__ __launch_bounds__(256) void k_adj_keys(int64_t K, const int32_t *__restrict__ ids, uint64_t *__restrict__ key,
                                                  int32_t *__restrict__ idx) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < K; i += (int64_t)gridDim.x * 256) {
        key[i] = (uint64_t)(ids[key[i]] - 1);
        idx[i] = (int32_t)i;
    }
}

__global__ __launch_bounds__(256) void k_adj_gids(int64_t K, const uint64_t *__restrict__ key, int32_t *__restrict__ gid) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < K; i += (int64_t)gridDim.x * 256) gid[i] = (int32_t)key[i];
}

static int bits_for(int64_t n) {  // of the numbers below n
    int b = 0;
    while (b < 32 && ((int64_t)1 << b) < n) ++b;
    return b;
}

size_t adjoint_group_scratch(int64_t K) { return group_scratch_bytes(K) + 20 * (size_t)K + 2048; }

hipError_t adjoint_values(int64_t K, const float *const coord[3], const float *df, int64_t max_groups, void *scratch,
                          size_t scratch_bytes, int32_t *counts, AdjValues *v, hipStream_t st) {
    v->K = K;
    v->free = Carve{(char *)scratch, scratch_bytes};
    v->count = counts;
    v->max_groups = max_groups;
    const float *const val[kFields] = {coord[0], coord[1], coord[2], df, nullptr, nullptr};
    if (!carve_fields(val, max_groups, v->free, v->f)) return hipErrorInvalidValue;
    return count_fields(K, v->f, counts, st);
}

hipError_t adjoint_groups(const AdjValues &v, const int32_t *cls, int32_t n_classes, int64_t max_cells,
                          int32_t *order, int32_t *gid, float4 *gtab, int32_t *gcls, int64_t *n_groups, hipStream_t st) {
    *n_groups = -1;
    const int64_t K = v.K;
    const Fields &f = v.f;
    const int32_t *count = v.count;
    Carve w = v.free;
    const int64_t cell_limit = max_cells < dense_cell_limit(K) ? max_cells : dense_cell_limit(K);
    AdjCells c{};
    c.n = c.C = n_classes;
    for (int q = 0; q < 4; ++q) {  // (a field has no more values than there are groups)
        if (count[q] > f.cap) return hipSuccess;
        c.nv[q] = f.val[q] ? count[q] : 1;
        c.shift[q] = rank_shift(count[q]);
        c.n *= c.nv[q];
        if (c.n > cell_limit) return hipSuccess;
    }
    hipError_t e;
    if ((e = rank_fields(f, count, st)) != hipSuccess) return e;
    c.flag = w.take<int32_t>((size_t)c.n);
    c.ids = w.take<int32_t>((size_t)c.n);
    uint64_t *key = w.take<uint64_t>(K), *sorted = w.take<uint64_t>(K);
    int32_t *idx = w.take<int32_t>(K);
    size_t b1 = 0, b2 = 0;
    if ((e = inclusive_sum(nullptr, &b1, (const int32_t *)nullptr, nullptr, c.n, st)) != hipSuccess) return e;
    if ((e = sort_pairs(nullptr, &b2, key, sorted, idx, order, K, 64, st)) != hipSuccess) return e;
    char *tmp = w.take<char>(b1 > b2 ? b1 : b2);
    if (!c.flag || !c.ids || !key || !sorted || !idx || !tmp) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zero_i32, grid_for(c.n), dim3(256), 0, st, c.n, c.flag);
    hipLaunchKernelGGL(k_adj_cells, grid_for(K), dim3(256), 0, st, K, f, c, cls, key);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = inclusive_sum(tmp, &b1, (const int32_t *)c.flag, c.ids, c.n, st)) != hipSuccess) return e;
    int32_t G = 0;
    if ((e = hipMemcpyAsync(&G, c.ids + (c.n - 1), sizeof(G), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    if (G > v.max_groups) return hipSuccess;
    hipLaunchKernelGGL(k_adj_tables, dim3((unsigned)((c.n + 255) / 256)), dim3(256), 0, st, f, c, gtab, gcls);
    hipLaunchKernelGGL(k_adj_keys, grid_for(K), dim3(256), 0, st, K, c.ids, key, idx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int bits = bits_for(G) < 1 ? 1 : bits_for(G);
    if ((e = sort_pairs(nullptr, &b2, key, sorted, idx, order, K, (unsigned)bits, st)) != hipSuccess) return e;
    if (b2 > w.left + (size_t)(w.p - tmp)) return hipErrorInvalidValue;
    if ((e = sort_pairs(tmp, &b2, key, sorted, idx, order, K, (unsigned)bits, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_adj_gids, grid_for(K), dim3(256), 0, st, K, sorted, gid);
    *n_groups = G;
    return hipGetLastError();
}

// ---- padded group-sorted layout ---------------------------------------------
// Isochromats are ordered by (x-group, z-group, index) and every run of equal
// (x-group, z-group), or piece of a long one, is padded to a multiple of 8 with copies of its first
// member carrying M0 = 0.  A thread's 8 (or 4) consecutive isochromats then always
// share both groups.  The sort takes the bits that the group counts need: 3
// passes of 8 bits instead of 8, for the 6.8 M isochromats above 0.2 ms
// instead of 0.65.
__global__ void k_pair_keys(int64_t K, const int32_t *__restrict__ gx, const int32_t *__restrict__ gz, int zbits,
                            uint64_t *__restrict__ key, int32_t *__restrict__ idx) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        key[i] = ((uint64_t)(uint32_t)gx[i] << zbits) | (gz ? (uint32_t)gz[i] : 0u);
        idx[i] = (int32_t)i;
    }
}

// rid = inclusive scan of the run starts (1-based); rstart and the run's groups.
// *cuts (zero before) += runs that go on with the key of the one before
__global__ void k_run_start(int64_t K, const uint64_t *__restrict__ key, int zbits, const int32_t *__restrict__ rid,
                            int32_t *__restrict__ rstart, int32_t *__restrict__ gx, int32_t *__restrict__ gz,
                            int32_t *__restrict__ cuts) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = rid[i] - 1;
        if (i == 0 || rid[i - 1] - 1 != r) {
            const uint64_t k = key[i];
            rstart[r] = (int32_t)i;
            gx[r] = (int32_t)(k >> zbits);
            gz[r] = (int32_t)(k & (((uint64_t)1 << zbits) - 1));
            if (i > 0 && key[i - 1] == k) atomicAdd(cuts, 1);
        }
    }
}

__global__ void k_run_plen(int64_t R, int64_t K, const int32_t *__restrict__ rstart, int32_t *__restrict__ plen) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t L = (int32_t)((r + 1 < R ? rstart[r + 1] : K) - rstart[r]);
        plen[r] = (L + 7) & ~7;  // 8-isochromat sweep threads never straddle a run
    }
}

static hipError_t sort_runs(Layout *l, const int32_t *gid_x, const int32_t *gid_z, int zbits, int bits, Carve w,
                            hipStream_t st) {
    uint64_t *key = w.take<uint64_t>(l->K), *key2 = w.take<uint64_t>(l->K);
    int32_t *idx = w.take<int32_t>(l->K);
    size_t b1 = 0, b2 = 0;
    hipError_t e;
    if ((e = sort_pairs(nullptr, &b1, key, key2, idx, l->order, l->K, (unsigned)bits, st)) != hipSuccess) return e;
    if ((e = inclusive_sum(nullptr, &b2, head_flags(key2, l->K), l->rid, l->K, st)) != hipSuccess) return e;
    char *tmp = w.take<char>(b1 > b2 ? b1 : b2);
    if (!key || !key2 || !idx || !tmp) return hipErrorInvalidValue;
    const dim3 g = grid_for(l->K);
    hipLaunchKernelGGL(k_pair_keys, g, dim3(256), 0, st, l->K, gid_x, gid_z, zbits, key, idx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sort_pairs(tmp, &b1, key, key2, idx, l->order, l->K, (unsigned)bits, st)) != hipSuccess) return e;
    if ((e = inclusive_sum(tmp, &b2, head_flags(key2, l->K), l->rid, l->K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, st, (int64_t)1, l->cuts);
    hipLaunchKernelGGL(k_run_start, g, dim3(256), 0, st, l->K, key2, zbits, l->rid, l->rstart, l->gx, l->gz, l->cuts);
    return hipGetLastError();
}

// Order and runs of the layout from natural-order x (and optional z) group ids
// of Gx and Gz groups: everything in *l (its arrays in the scratch), which
// synchronizes the stream twice, for the number of runs and the padded count.
hipError_t build_layout(int64_t K, const int32_t *gid_x, int64_t Gx, const int32_t *gid_z, int64_t Gz, void *scratch,
                        size_t scratch_bytes, Layout *l, hipStream_t st) {
    Carve w{(char *)scratch, scratch_bytes};
    l->K = K;
    int32_t **arr[] = {&l->order, &l->rid, &l->rstart, &l->pstart, &l->plen, &l->gx, &l->gz};
    for (int32_t **a : arr)
        if (!(*a = w.take<int32_t>(K))) return hipErrorInvalidValue;
    if (!(l->cuts = w.take<int32_t>(1))) return hipErrorInvalidValue;
    const int zbits = gid_z ? bits_for(Gz) : 0, bits = zbits + bits_for(Gx);
    hipError_t e = sort_runs(l, gid_x, gid_z, zbits, bits < 1 ? 1 : bits, w, st);
    if (e != hipSuccess) return e;
    int32_t R = 0, cuts = 0;
    if ((e = hipMemcpyAsync(&R, l->rid + (K - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(&cuts, l->cuts, sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    l->R = R;
    l->pairs = R - cuts;
    l->free = w;
    hipLaunchKernelGGL(k_run_plen, grid_for(R), dim3(256), 0, st, (int64_t)R, K, l->rstart, l->plen);
    size_t b = 0;
    if ((e = exclusive_sum(nullptr, &b, l->plen, l->pstart, R, st)) != hipSuccess) return e;
    char *tmp = w.take<char>(b);
    if (!tmp) return hipErrorInvalidValue;
    if ((e = exclusive_sum(tmp, &b, l->plen, l->pstart, R, st)) != hipSuccess) return e;
    int32_t last[2] = {0, 0};
    if ((e = hipMemcpyAsync(&last[0], l->pstart + (R - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipMemcpyAsync(&last[1], l->plen + (R - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    l->kint = (int64_t)last[0] + last[1];
    return hipSuccess;
}

// A run's slot: its rank by its first isochromat in the caller's order (the
// sort is stable: that one comes first).
__global__ void k_first_flags(int64_t R, const int32_t *__restrict__ rstart, const int32_t *__restrict__ order,
                              int32_t *__restrict__ flag) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x)
        flag[order[rstart[r]]] = 1;
}

__global__ void k_run_slots(int64_t R, const int32_t *__restrict__ rstart, const int32_t *__restrict__ order,
                            const int32_t *__restrict__ rank, int32_t *__restrict__ slot) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (int64_t)gridDim.x * blockDim.x)
        slot[r] = rank[order[rstart[r]]];
}

hipError_t place_runs(const Layout &l, int32_t *slot, hipStream_t st) {
    Carve w = l.free;
    int32_t *flag = w.take<int32_t>(l.K), *rank = w.take<int32_t>(l.K);
    size_t b = 0;
    hipError_t e = exclusive_sum(nullptr, &b, flag, rank, l.K, st);
    if (e != hipSuccess) return e;
    char *tmp = w.take<char>(b);
    if (!flag || !rank || !tmp) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zero_i32, grid_for(l.K), dim3(256), 0, st, l.K, flag);
    hipLaunchKernelGGL(k_first_flags, grid_for(l.R), dim3(256), 0, st, l.R, l.rstart, l.order, flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = exclusive_sum(tmp, &b, flag, rank, l.K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_run_slots, grid_for(l.R), dim3(256), 0, st, l.R, l.rstart, l.order, rank, slot);
    return hipGetLastError();
}

// What the members of a run share comes from the group tables (x, T1, T2, dB0;
// z where z is grouped) and is written by k_place, in sorted order: streams.
// M0, y, the y-group and the inverse lists go between the layout and the
// caller's order, a column of the phantom at a time: a cache line of the
// caller's arrays holds neighbours that the layout places a whole column
// apart.  So each has a pass of its own (k_move), and the passes give every
// die a contiguous part of the layout: the lines of one column and one array
// (1.7 MB of a 512 x 512 x 26 grid) can stay in its L2 until the next columns
// have used the rest of them.  Measured with the 6.8 M isochromats above: 57 us
// and 5 times 48 us; all in one pass over blocks in launch order, with the
// lines of five arrays coming from beyond the L2 once per element, 445 us.
__device__ __forceinline__ void write_position(const LayoutOut &o, int64_t pos, int32_t k, bool pad, int32_t gx,
                                               int32_t gz) {
    const float4 g = o.gtab_x[gx];
    o.perm[pos] = pad ? -1 : k;
    o.x[pos] = g.x;
    if (o.gtab_z) o.z[pos] = o.gtab_z[gz].x;
    o.t1[pos] = g.y;
    o.t2[pos] = g.z;
    o.df[pos] = g.w;
    o.gid_x[pos] = gx;
    if (o.gid_z) o.gid_z[pos] = gz;
}

__global__ __launch_bounds__(256) void k_place(Layout l, LayoutOut o) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < l.K; i += (int64_t)gridDim.x * 256) {
        const int32_t r = l.rid[i] - 1, k = l.order[i];
        const int64_t pos = (int64_t)l.pstart[r] + (i - l.rstart[r]);
        write_position(o, pos, k, false, l.gx[r], l.gz[r]);
        if (o.run_of4 && (pos & 3) == 0) o.run_of4[pos >> 2] = r;
    }
}

// kMove: dst[pos] <- src[perm[pos]]; kInverse: dst[perm[pos]] <- pos; kRunOf:
// dst[perm[pos]] <- slot of the position's run.  Padding is left out.
enum { kMove, kInverse, kRunOf };

template <int OP>
__global__ __launch_bounds__(256) void k_move(int64_t n4, int32_t per_die, const int4 *__restrict__ perm4,
                                              const int32_t *__restrict__ src, const int32_t *__restrict__ run_of4,
                                              int32_t *__restrict__ dst) {
    // workgroups go to the 8 dies in turn: die d takes the blocks d per_die, d per_die + 1, ...
    const int64_t q = ((int64_t)(blockIdx.x & 7) * per_die + (blockIdx.x >> 3)) * 256 + threadIdx.x;
    if (q >= n4) return;
    const int4 p = perm4[q];
    const int32_t k[4] = {p.x, p.y, p.z, p.w};
    if (OP == kMove) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k[j] >= 0) dst[4 * q + j] = src[k[j]];
    } else {
        const int32_t s = OP == kRunOf ? src[run_of4[q]] : 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k[j] >= 0) dst[k[j]] = OP == kRunOf ? s : (int32_t)(4 * q + j);
    }
}

__device__ __forceinline__ void write_padding(const LayoutOut &o, int64_t pos, int32_t k, int32_t gx, int32_t gz) {
    write_position(o, pos, k, true, gx, gz);
    o.y[pos] = o.ph.y[k];
    if (!o.gtab_z) o.z[pos] = o.ph.z[k];
    o.m0[pos] = 0.0f;
    if (o.gid_y) o.gid_y[pos] = o.nat_y[k];
}

// Padding: 8 threads per run for its last 8 positions (fewer than 8 of them are
// padding), then the positions behind the last run, which copy isochromat 0;
// and the arrays per run.
__global__ __launch_bounds__(256) void k_pad(Layout l, LayoutOut o) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, r = t >> 3;
    if (r >= l.R) {
        const int64_t pos = l.kint + (t - 8 * l.R);
        if (pos < o.Kpad) write_padding(o, pos, 0, o.nat_x[0], o.nat_z ? o.nat_z[0] : 0);
        if (t == 8 * l.R && o.run_first4) o.run_first4[l.R] = (int32_t)(l.kint >> 2);
        return;
    }
    const int32_t p0 = l.pstart[r], s0 = l.rstart[r];
    const int32_t L = (int32_t)((r + 1 < l.R ? l.rstart[r + 1] : l.K) - s0);
    const int64_t j = l.plen[r] - 8 + (t & 7), pos = p0 + j;
    if (j >= L) {
        write_padding(o, pos, l.order[s0], l.gx[r], l.gz[r]);
        if (o.run_of4 && (pos & 3) == 0) o.run_of4[pos >> 2] = (int32_t)r;
    }
    if ((t & 7) == 0 && o.run_first4) {
        o.run_first4[r] = p0 >> 2;
        o.run_gx[r] = l.gx[r];
        o.run_gz[r] = l.gz[r];
    }
}

hipError_t write_layout(const Layout &l, const LayoutOut &o, hipStream_t st) {
    hipLaunchKernelGGL(k_place, grid_for(l.K), dim3(256), 0, st, l, o);
    const int64_t n = 8 * l.R + (o.Kpad - l.kint) + 1;
    hipLaunchKernelGGL(k_pad, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, l, o);
    const int64_t n4 = l.kint / 4;
    const int32_t per_die = (int32_t)((n4 + 2047) / 2048);
    const int4 *perm4 = (const int4 *)o.perm;
    auto gather = [&](const void *src, void *dst) {
        hipLaunchKernelGGL(k_move<kMove>, dim3(8 * per_die), dim3(256), 0, st, n4, per_die, perm4, (const int32_t *)src,
                           (const int32_t *)nullptr, (int32_t *)dst);
    };
    gather(o.ph.y, o.y);
    gather(o.ph.m0, o.m0);
    if (!o.gtab_z) gather(o.ph.z, o.z);
    if (o.gid_y) gather(o.nat_y, o.gid_y);
    hipLaunchKernelGGL(k_move<kInverse>, dim3(8 * per_die), dim3(256), 0, st, n4, per_die, perm4,
                       (const int32_t *)nullptr, (const int32_t *)nullptr, o.inv);
    if (o.run_of)
        hipLaunchKernelGGL(k_move<kRunOf>, dim3(8 * per_die), dim3(256), 0, st, n4, per_die, perm4, o.slot,
                           (const int32_t *)o.run_of4, o.run_of);
    return hipGetLastError();
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

hipError_t group_runs(const Layout &l, int64_t n_groups, int32_t **xrun, hipStream_t st) {
    Carve w = l.free;
    if (!(*xrun = w.take<int32_t>((size_t)n_groups + 1))) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_group_runs, grid_for(l.R + 1), dim3(256), 0, st, l.R, l.gx, n_groups, *xrun);
    return hipGetLastError();
}

size_t group_scratch_bytes(int64_t K) {
    size_t b[3] = {0, 0, 0};
    const int64_t n = dense_cell_limit(K);  // >= K
    const bool sized =
        sort_pairs(nullptr, &b[0], nullptr, nullptr, nullptr, nullptr, K, 64, 0) == hipSuccess &&
        inclusive_sum(nullptr, &b[1], (const int32_t *)nullptr, nullptr, n, 0) == hipSuccess &&
        exclusive_sum(nullptr, &b[2], nullptr, nullptr, n, 0) == hipSuccess;
    size_t tmp = 0;
    for (size_t v : b) tmp = v > tmp ? v : tmp;
    // a failed size query leaves generous room; the sorts and scans report their own errors
    if (!sized) tmp = ((size_t)64 << 20) + 16 * (size_t)K;
    // the largest of group_axis (4 u64 + 4 i32 arrays), build_layout (2 u64 + 8 i32)
    // and dense_groups (2 i32 per cell and the field tables), plus tmp
    const size_t sorted = 48 * (size_t)K, dense = 8 * (size_t)n + 4 * (kFieldCounts + kFieldTables + kFieldFound);
    return (sorted > dense ? sorted : dense) + tmp + 17 * 256;
}

// Group one axis by sorting, ids in the order of (coord, T1, T2, df) or, with
// coord_last, (T1, T2, df, coord): the z-groups of one tissue then are
// neighbours, and so are the transition rows that the runs of an x-group read
// (one tissue, successive z).  coord = r_a of every isochromat (natural order).
// Writes gid_nat[K] (natural order) and returns the group count through
// *n_groups (synchronizes the stream); sorted_table then writes gtab[n_groups]
// = (coord, T1, T2, df) while the scratch holds.
hipError_t group_axis(int64_t K, bool coord_last, const float *coord, const float *t1, const float *t2, const float *df,
                      void *scratch, size_t scratch_bytes, int32_t *gid_nat, SortedAxis *s, int64_t *n_groups,
                      hipStream_t st) {
    Carve w{(char *)scratch, scratch_bytes};
    uint64_t *hi = w.take<uint64_t>(K), *lo = w.take<uint64_t>(K), *k2 = w.take<uint64_t>(K), *k3 = w.take<uint64_t>(K);
    int32_t *idx0 = w.take<int32_t>(K), *idx1 = w.take<int32_t>(K), *flag = w.take<int32_t>(K),
            *order = w.take<int32_t>(K);
    if (!order) return hipErrorInvalidValue;
    void *tmp = w.p;
    size_t tmp_bytes = w.left;
    const dim3 g = grid_for(K);
    hipError_t e;
    if (coord_last)
        hipLaunchKernelGGL(k_keys, g, dim3(256), 0, st, K, t1, t2, df, coord, hi, lo, idx0);
    else
        hipLaunchKernelGGL(k_keys, g, dim3(256), 0, st, K, coord, t1, t2, df, hi, lo, idx0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // LSD: low half first (carry indices), then the high half of the same records.
    if ((e = sort_pairs(tmp, &tmp_bytes, lo, k2, idx0, idx1, K, 64, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_gather_u64, g, dim3(256), 0, st, K, hi, idx1, k3);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sort_pairs(tmp, &tmp_bytes, k3, hi, idx1, order, K, 64, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_gather_u64, g, dim3(256), 0, st, K, lo, order, k2);  // low half in final order
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_heads, g, dim3(256), 0, st, K, hi, k2, flag);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = inclusive_sum(tmp, &tmp_bytes, (const int32_t *)flag, idx0, K, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_assign, g, dim3(256), 0, st, K, idx0, order, gid_nat);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int32_t last = 0;
    if ((e = hipMemcpyAsync(&last, idx0 + (K - 1), sizeof(int32_t), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    *s = SortedAxis{idx0, order};
    *n_groups = last;
    return hipSuccess;
}

hipError_t sorted_table(int64_t K, const SortedAxis &s, const float *coord, const float *t1, const float *t2,
                        const float *df, float4 *gtab, hipStream_t st) {
    hipLaunchKernelGGL(k_group_table, grid_for(K), dim3(256), 0, st, K, s.ids, s.order, coord, t1, t2, df, gtab);
    return hipGetLastError();
}

}  // namespace gbs
