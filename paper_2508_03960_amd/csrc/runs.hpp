// Grouped simulation per run of the layout (k_runs.hip).
//
// A run of the group-sorted layout holds isochromats of equal (x, z, T1, T2,
// dB0), up to 3 kRunPiece - 2 of them.  When a simulation starts from (0, 0, M0) and no B1 = 0 map before
// a transition carries a y moment, the members of a run differ in nothing
// that moves M / M0: all of them keep one ratio m_r, so each run is stepped
// once.  The group sums of a with-ADC subsequence (Eq. 9) become
//   S_g = sum over the runs r of x-group g of f_r m_r Y_r(c),
//   Y_r(c) = sum over the members k of r of S(k, p) M0_k exp(-2 pi i c y_k),
// with f_r the x- and z-group factors of its map and c its y moment.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gbs {

// y phase coefficients (cycles per metre) of the emissions on a grid:
// line l stands for c0 + d (l - n/2 + 1/2), l < n = 32 nb.
struct YLines {
    double c0, d;
    int32_t nb;       // b magnitudes; 32 lines each
    int32_t n_lines;  // 32 nb
};

constexpr int64_t kRunMaxRuns = UINT32_MAX / 48;  // 48-byte rows at 32-bit offsets
constexpr int64_t kRunMaxSlots = (int64_t)1 << 30;  // 4-byte slots at 32-bit offsets
constexpr int kRunTile = 8;      // runs per row of the Y layout
constexpr int kRunLinesSet = 256;  // lines of one 16 x 16 pair of tiles

// Y[coil][run / kRunTile][line][run % kRunTile] for the runs [r0, r0 + n) (r0 a
// multiple of kRunTile), stored from run r0 on.
struct RunYArgs {
    int64_t r0, n, n_runs;
    const int32_t *first4;  // first 4-slot quad of each run, n_runs + 1 entries
    const float *y, *m0;    // layout order (padding: M0 = 0)
    const float *coil;      // planes re, im per coil of coil_plane floats, or null
    int64_t coil_plane;
    int32_t n_coils;
    YLines lines;
    float2 *out;
    int64_t out_coil;  // float2 entries per coil
};

// One grouped operation as the run sweep reads it (see SweepOp).  Every table
// pointer is valid: an operation without one points at an identity row, with
// its bit of `flags` (kRun...) clear, so that the lanes all read that row and
// every operation issues the same loads.
enum { kRunPreX = 1 << 16, kRunPreZ = 1 << 17, kRunRows = 1 << 18, kRunEmitZ = 1 << 19 };
struct RunOp {
    int32_t flags;    // kOpPre, kOpRf, kOpEmit, kPreMz, kRun...
    int32_t rf_axis;  // rows per x-group (0), z-group (2) or run (kPairRows)
    int32_t line;         // emission: its line of Y
    int32_t gsum_stride;  // coil p sums at gsum + p gsum_stride
    const float4 *pre_xtab;
    const float2 *pre_ztab;
    const float4 *ttab;
    const float4 *emit_xtab;
    const float2 *emit_ztab;
    double2 *gsum;
};
// Identity rows: a factor 1 with E1 = 1, and a transition's three rows.
constexpr float kRunIdentity[16] = {1, 0, 1, 0, 1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0};

// Operations [first, first + n) of the list; emit_only: they only emit.
struct RunPart {
    int32_t first, n, emit_only;
};
constexpr int kRunMaxParts = 6;

struct RunSweepArgs {
    int64_t r0;              // first run of the batch (Y starts there)
    int64_t n_runs;
    const int32_t *first;    // wavefront w of the launch takes the runs [first[w], first[w + 1]), at most 64
    int32_t n_waves;
    const int32_t *gx, *gz, *slot;  // groups, and the place of the ratio in m, per run
    const RunOp *ops;
    RunPart parts[kRunMaxParts];
    int32_t n_parts;
    int32_t n_coils;
    const float2 *y;   // as written by launch_run_y for the same runs
    int32_t n_lines;
    int64_t y_coil;
    float4 *m;         // final (mx, my, mz, 0) / M0 of all runs
};

// M_k = M0_k m_r e^{-2 pi i cy y_k} (transverse) in the caller's order.
struct RunStateArgs {
    int64_t K;
    const int32_t *run;  // place of the ratio of isochromat k's run in m
    const float *m0, *y;
    double cy;
    const float4 *m;
    float *ox, *oy, *oz;
};

hipError_t launch_run_y(const RunYArgs &a, hipStream_t st);
hipError_t launch_run_sweep(const RunSweepArgs &a, hipStream_t st);
hipError_t launch_run_state(const RunStateArgs &a, hipStream_t st);

}  // namespace gbs
