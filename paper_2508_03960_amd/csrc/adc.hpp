// ADC samples from group sums (Eq. 8 with Eq. 10) for readouts whose sample
// times and gradient moments are arithmetic in the sample index.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace gbs {

// Sample n of the block is taken at tau0 + n dtau after the block start, with
// gamma_bar * (gradient moment since the block start) = cyc0 + n dcyc.
struct AdcLinJob {
    int32_t n_samples;
    int32_t n_groups;
    const double2 *gsum;
    const float4 *gtab;  // (coord, T1, T2, df) per group
    double tau0, dtau;
    double cyc0, dcyc;
    int64_t sig_offset;
};

// The readouts of equal sample times, moments and groups (the echoes and shots
// of a repeated timing, and the coils) as one matrix product: rows are
// readouts, the inner dimension their groups, columns the samples.
struct AdcClass {
    double tau0, dtau, cyc0, dcyc;  // as AdcLinJob
    const float4 *gtab;
    int32_t n_groups, n_samples;
    int32_t split;    // groups per workgroup, a multiple of kAdcMmSub up to kAdcMmSplit
    int32_t n_split;  // ceil(n_groups / split)
};
struct AdcRow {
    const double2 *gsum;
    int64_t sig_offset;
    int64_t part, stride;  // first entry of the row in the first split's partial sums, and from split to split
    int32_t cls, pad;
};
struct AdcTile {  // rows [row, row + n_rows) of one class, samples from n0 on
    int32_t cls, row, n_rows, n0;
};
// Tiles [tile0, tile0 + n_tiles) and their rows in one launch, n_part partial sums.
struct AdcBatch {
    int32_t tile0, n_tiles, row0, n_rows, max_split, max_samples;
    int64_t n_part;
};
// Partial sums of one launch: all of a 27M FSE (42 MB, with 8 coils in two); a
// timing whose tiles alone take more is evaluated one by one.
constexpr size_t kAdcPartCap = (size_t)256 << 20;
constexpr int kAdcMmRows = 64;    // rows per workgroup
constexpr int kAdcMmCols = 128;   // samples per workgroup
constexpr int kAdcMmSub = 32;     // groups staged at a time
constexpr int kAdcMmSplit = 224;  // most groups per workgroup, 32 at a time (k_adc_lin: 28 per thread, 8 threads)
// Rows that a tile needs: its cost is that of 64 rows.  us for a tile of 64 by the
// product and for r rows by k_adc_lin: 400000 groups, 64 samples 270 and 6.8 r,
// 128 samples 290 and 9.5 r, 256 samples 550 and 15.8 r; 60000 groups 64 and 1.2 r,
// 69 and 1.65 r, 120 and 2.7 r.  Rows that fill no tile are evaluated one by one.
__host__ __device__ constexpr int adc_mm_min_rows(int n_samples) { return n_samples <= 64 ? 56 : 48; }
// Terms (rows x samples x groups) from which the product is the faster one: 97 x 131
// x 8700 take 42 us either way, 32 x 64 x 700 take 8.9 us in k_adc_lin's one
// launch and 12 us in the product's two.
constexpr double kAdcMmMinTerms = 1.5e8;

// part[row.part + split * row.stride + n] <- the partial sums (FP32), then
// sig += their FP64 sums
hipError_t launch_adc_mm(const AdcClass *cls, const AdcRow *rows, const AdcTile *tiles, const AdcBatch &b, float2 *part,
                         double *sig, hipStream_t st);

hipError_t launch_adc_lin(const AdcLinJob *jobs, int n_jobs, int max_groups, double *sig, hipStream_t st);

}  // namespace gbs
