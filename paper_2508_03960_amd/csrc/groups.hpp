// Device grouping helpers (k_groups.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kernels.hpp"

namespace gbs {

constexpr int kFields = 6;  // x, y, z, T1, T2, dB0
constexpr int kFieldCap = 8192;  // distinct values of a field up to which phantoms are grouped without a sort
constexpr int kFieldSlots = 2 * kFieldCap;
constexpr int kRunPiece = 512;  // isochromats: runs of twice as many and more are cut into pieces

// Pieces of the grouping scratch, 256-byte aligned (null when it is used up).
struct Carve {
    char *p;
    size_t left;
    template <typename T>
    T *take(size_t n) {
        const size_t b = (n * sizeof(T) + 255) & ~(size_t)255;
        if (b > left) {
            left = 0;
            return nullptr;
        }
        T *r = (T *)p;
        p += b;
        left -= b;
        return r;
    }
};

struct Fields {
    const float *val[kFields];  // null: not needed
    uint32_t *set[kFields];     // [kFieldSlots] hash table of the values, zero before k_field_values
    uint32_t *list[kFields];    // [kFieldCap] distinct values as found
    uint32_t *sorted[kFields];  // [kFieldCap] in ascending order
    uint64_t *rank[kFields];    // [kFieldSlots] (value << 32 | rank), zero before k_field_ranks
    int32_t cap;                // values of a field from beyond which it is given up
    int32_t *count;             // [kFields], 0 or given up before k_field_values
};

// Cells: axis a's block [base[a], base[a + 1]) of the products coordinate x
// tissue (z: tissue x coordinate), then one cell per tissue, a tissue being
// (rank T1, rank T2, rank dB0).
struct Cells {
    int64_t base[5];
    int32_t nc[3], n2, nd, nt;  // values per coordinate (0: axis not grouped), of T2 and dB0; tissues
    int32_t shift[kFields];     // of the rank tables
    int32_t *flag, *ids;        // occupied cells, and their inclusive sum
    int32_t *gid[3];            // natural order: the cell, then the group
};

struct DenseGroups {
    Fields f;
    Cells c;
    int32_t *d_total;
    int32_t total[4];  // groups of x; of x and y; of all axes; of all axes and the tissues
};

struct SortedAxis {
    const int32_t *ids, *order;  // 1-based group per sorted position, its isochromat
};

// The padded layout's order and runs (arrays in the grouping scratch).
struct Layout {
    int64_t K, R, kint;  // isochromats, runs, padded count (a multiple of 8)
    int64_t pairs;       // (x-group, z-group) pairs: the runs less the cuts of long ones
    int32_t *order;      // [K] isochromats by (x-group, z-group, index)
    int32_t *rid;        // [K] their run, 1-based
    int32_t *rstart, *pstart, *plen;  // [R] first sorted and first padded position, padded length
    int32_t *gx, *gz;    // [R] groups
    int32_t *cuts;       // runs that go on with the pair of the one before
    Carve free;          // the rest of the scratch
};

struct LayoutOut {
    int64_t Kpad;
    PhantomPtrs ph;
    const float4 *gtab_x, *gtab_z;              // gtab_z null: no z-groups
    const int32_t *nat_x, *nat_y, *nat_z;       // groups in natural order (y, z: or null)
    int32_t *perm, *inv;                        // perm: -1 at padding
    float *x, *y, *z, *t1, *t2, *df, *m0;       // [Kpad]
    int32_t *gid_x, *gid_y, *gid_z;             // [Kpad] (y, z: or null)
    const int32_t *slot;                        // [R]
    int32_t *run_of4, *run_of;                  // run per quad, slot per isochromat (or both null)
    int32_t *run_first4, *run_gx, *run_gz;      // per run: first quad (and kint / 4 after the last), groups (or all null)
};

size_t group_scratch_bytes(int64_t K);
hipError_t dense_groups(int64_t K, const float *const coord[3], const float *t1, const float *t2, const float *df,
                        void *scratch, size_t scratch_bytes, int32_t *const gid[3], DenseGroups *d, bool *done,
                        hipStream_t st);
hipError_t dense_tables(const DenseGroups &d, float4 *const gtab[3], float4 *ttab, int32_t *tmap, hipStream_t st);
// Groups of the adjoint: isochromats of equal coord[a] (null: not compared),
// dB0 and class, in that order.
// adjoint_values collects the values of the coordinates and dB0 in the scratch
// (adjoint_group_scratch bytes) and copies their counts to the pinned counts.
// After the stream has been waited for, adjoint_groups writes order and gid[K]
// (isochromats sorted by group, their groups), and per group (coordinates or 0,
// dB0) and the class; *n_groups = -1: too many distinct values, more than
// max_cells products of them, or more than max_groups groups.  It synchronizes
// the stream.
struct AdjValues {
    int64_t K;
    Fields f;
    Carve free;  // the rest of the scratch
    const int32_t *count;
    int64_t max_groups;
};
size_t adjoint_group_scratch(int64_t K);
hipError_t adjoint_values(int64_t K, const float *const coord[3], const float *df, int64_t max_groups, void *scratch,
                          size_t scratch_bytes, int32_t *counts, AdjValues *v, hipStream_t st);
hipError_t adjoint_groups(const AdjValues &v, const int32_t *cls, int32_t n_classes, int64_t max_cells,
                          int32_t *order, int32_t *gid, float4 *gtab, int32_t *gcls, int64_t *n_groups, hipStream_t st);
hipError_t group_axis(int64_t K, bool coord_last, const float *coord, const float *t1, const float *t2, const float *df,
                      void *scratch, size_t scratch_bytes, int32_t *gid_nat, SortedAxis *s, int64_t *n_groups,
                      hipStream_t st);
hipError_t sorted_table(int64_t K, const SortedAxis &s, const float *coord, const float *t1, const float *t2,
                        const float *df, float4 *gtab, hipStream_t st);
hipError_t build_layout(int64_t K, const int32_t *gid_x, int64_t Gx, const int32_t *gid_z, int64_t Gz, void *scratch,
                        size_t scratch_bytes, Layout *l, hipStream_t st);
hipError_t place_runs(const Layout &l, int32_t *slot, hipStream_t st);
hipError_t write_layout(const Layout &l, const LayoutOut &o, hipStream_t st);
// first run of every x-group and the number of runs: [n_groups + 1] in the layout's scratch
hipError_t group_runs(const Layout &l, int64_t n_groups, int32_t **xrun, hipStream_t st);
// dst[i] <- src[perm[i]], 0 where perm[i] < 0 (layout padding), for i < n
hipError_t launch_gather_padded(int64_t n, const int32_t *perm, const float *src, float *dst, hipStream_t st);
// *bad <- 1 if any of a[0 .. n) is NaN or infinite (*bad is not cleared)
hipError_t launch_check_finite(int64_t n, const float *a, int *bad, hipStream_t st);
// dst row g (12 doubles) <- src row map[g], for g < n
hipError_t launch_expand_rows(const double *src, const int32_t *map, int64_t n, double *dst, hipStream_t st);

}  // namespace gbs
