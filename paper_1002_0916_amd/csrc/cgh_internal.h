// Internal declarations shared by the library's HIP sources (not installed).
//
// Workspace layout, point-record formats and the launch wrappers of every
// kernel.  All kernels target gfx950 (CDNA4, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace cgh {

constexpr int kWave = 64;
constexpr int kXcds = 8;

// MI355X dispatches workgroups round-robin over its 8 XCDs (linear id i runs
// on XCD i % 8), each with its own L2.  xcd_tile renumbers linear id i of n
// so that every XCD receives one contiguous range of tile indices: tiles
// that are neighbours in tile order (and share input data) then share an L2.
// A bijection on [0, n) for any n.
__device__ __forceinline__ unsigned xcd_tile(unsigned i, unsigned n) {
  const unsigned per = n / kXcds, rem = n % kXcds;
  const unsigned x = i % kXcds, k = i / kXcds;
  return x < rem ? x * (per + 1) + k : rem * (per + 1) + (x - rem) * per + k;
}

// Wave priority by progress.  The SIMD arbiter issues the oldest ready wave
// first, so the workgroups that share a CU from the launch on do not advance
// together: the first finishes long before the last, which then runs with few
// waves per SIMD.  A wave that starts at priority 3 and drops to 2, 1 and 0 as
// it passes each quarter of its loop yields to the waves behind it, so the
// workgroups of a CU finish close together.  Scheduling only: results do not
// change.  priority_step(i, n) is called at step i of a loop whose counter
// steps by one through [0, n).
__device__ __forceinline__ void priority_start() { __builtin_amdgcn_s_setprio(3); }
__device__ __forceinline__ void priority_step(int i, int n) {
  if (i == n / 4) __builtin_amdgcn_s_setprio(2);
  if (i == n / 2) __builtin_amdgcn_s_setprio(1);
  if (i == 3 * n / 4) __builtin_amdgcn_s_setprio(0);
}

// Workgroups of `threads` covering `count` items on a 1-D grid, or 0 when
// that exceeds the grid's x limit (2^31 - 1); launchers then return
// hipErrorInvalidValue instead of launching a truncated grid.
inline unsigned grid_blocks(int64_t count, int threads) {
  const int64_t b = (count + threads - 1) / threads;
  return (b < 1 || b > 0x7fffffff) ? 0u : (unsigned)b;
}

// ---------------------------------------------------------------- forward --
// The plain and compensated direct forwards stage kTile points at a time in LDS.
// The point arrays in the workspace are padded to a multiple of kPointPad with
// zero-amplitude points.
constexpr int kTile = 64;
constexpr int kTilePitch = kWave + 1;

// Compensated forward: a workgroup of kCompWaves waves covers 64 columns x
// (kCompWaves * kCompRows) rows; each wave owns kCompRows rows.  Its x-phases,
// row phases and amplitudes are staged in LDS a tile of kTile points at a
// time (x-phase rows padded to kTilePitch floats, so that lane-per-point
// writes hit distinct banks).  Overridable at build time for tuning
// experiments.
#ifndef CGH_COMP_WAVES
#define CGH_COMP_WAVES 8
#endif
#ifndef CGH_COMP_ROWS
#define CGH_COMP_ROWS 4
#endif
constexpr int kCompWaves = CGH_COMP_WAVES;
constexpr int kCompRows = CGH_COMP_ROWS;
constexpr int kCompThreads = kCompWaves * kWave;
constexpr int kCompRowsPerWG = kCompWaves * kCompRows;
static_assert(kWave % kCompWaves == 0, "x-phase fill splits the 64 columns over the waves");
static_assert(kTile % 16 == 0, "the inner loop takes 16 points per iteration");
// The compensated forward reads its x-phases from a column table
// [fwd_gx * 64][npad] while that takes at most kCompColTabMaxBytes; else it
// takes the points in chunks whose tables fit the row table's region, or forms
// the x-phases in the kernel (the same values).  Every row block of workgroups
// reads the table again, from the 256 MB Infinity Cache while it fits.
constexpr int64_t kCompColTabMaxBytes = int64_t(256) << 20;
constexpr int kPointPad = 64;

// ---------------------------------------------------------------- adjoint --
// An adjoint wave holds 64 points (one per lane) and sweeps a run of
// strip-rows: the hologram is cut into strips of kAdjCols columns, and the
// strip-rows (strip-major: strip s, row r -> s * ny + r) of every point group
// are split into equal contiguous runs, one per wave.  G is broadcast to the
// wave through scalar loads, one strip row at a time.
constexpr int kAdjCols = 32;
// Phase arithmetic of the adjoint kernel (Plan::adj_kind): the plain FP32
// phase, the compensated axis phases, or the recurrence of Eq. (2) along the
// strip row.  The compensated kind reads the cosine and sine of each row's
// y-phase from a table [ny][npad] and each strip column's x-phase from a table
// [nsx * kAdjCols][npad], both built by one precompute launch (the same
// values it would form itself, once per row or column and point instead of
// once per strip and point); when either table would exceed
// kAdjRowTabMaxBytes the kernel forms them inline instead
// (kAdjCompensatedInline: the same values, so the same result whenever the
// launch takes the same run count; its lower occupancy can give it another).
constexpr int kAdjPlain = 0;
constexpr int kAdjCompensated = 1;
constexpr int kAdjRecurrence = 2;
constexpr int kAdjCompensatedInline = 3;
constexpr int64_t kAdjRowTabMaxBytes = int64_t(512) << 20;
constexpr int kAdjThreads = kWave;
// At launch the number of runs is chosen so that kAdjRounds rounds of
// resident waves (CUs x resident waves per CU, from the occupancy query)
// cover the whole hologram with equal work per wave, and runs hold at least
// kAdjMinRun strip-rows.  The partial-sum buffer is sized for kAdjRounds
// rounds at up to 8 resident waves per SIMD on 256 CUs (kAdjMaxWaves), so
// the last round is never cut short at any occupancy a kernel reaches.
#ifndef CGH_ADJ_ROUNDS
#define CGH_ADJ_ROUNDS 3
#endif
constexpr int kAdjRounds = CGH_ADJ_ROUNDS;
constexpr int kAdjMaxWaves = kAdjRounds * 256 * 4 * 8;
constexpr int kAdjMinRun = 8;
// The adjoint's finalize spreads its partial planes over kAdjFinSlices threads
// for each of kAdjFinPoints points per workgroup.
constexpr int kAdjFinPoints = 16;
constexpr int kAdjFinSlices = 64;

// The adjoint's order of strip-rows.  The (strip, row) space is cut into
// kXcds blocks, H strip groups x B row bands (H B = kXcds): block
// beta = h B + b covers strips [h sh, min(nsx, (h + 1) sh)) and rows
// [b br, min(ny, (b + 1) br)), strip-major inside, and off[beta] is its first
// index in the order (off[kXcds] = nsx ny).  Runs are equal ranges of this
// order and xcd_tile places consecutive runs on one XCD, so each XCD works
// through about one block: it reads only its band of the row table and its
// strips' share of the column table.  H is chosen to minimise the bytes the
// XCDs read between them: H row tables and B column tables.
struct AdjOrder {
  int64_t off[kXcds + 1];
  int sh, br, B;
};

// Point records, all produced on the device by the prep kernel from the FP32
// inputs with FP64 arithmetic.
//
//  plain   float4 {x, y, Prev, A}         Prev = fl32(p^2 / (2 lambda z)),
//                                           the phase coefficient in
//                                           revolutions per pixel^2.
//  axis    float[8] {c, Ph, Pl, b, d, A, v, 0} per axis (x then y arrays):
//          c = rint(v) (v = x_j or y_j), f = v - c (exact),
//          Ph = fl32(Prev), Pl = fl32(Prev - Ph),
//          b = fl32(-2 Prev f), d = fl32(Prev f^2),
//          so that Prev (h - v)^2 = (Ph + Pl) m^2 + b m + d with m = h - c,
//          an integer: m^2 is exact in FP32 for |m| < 4096.
//  f64     double4 {x, y, Prev, A}.
constexpr int kAxisRec = 8;

struct Workspace {
  float4* plain;   // [npad]
  float* amp;      // [npad] amplitudes A_j (contiguous, for scalar loads)
  float* xrec;     // [npad][8]
  float* yrec;     // [npad][8]
  double4* rec64;  // [npad]
  double* tab64;   // FP64 forward: y then x tables of a chunk of points
  double* planes64;  // FP64 forward: partial sums [f64_slices][ny][nx]
  float* ytab;     // forward, compensated: [groups][npad][kCompRows]
  float* xtab;     // forward, compensated (optional): [fwd_gx * 64][npad] x-phases
  float* planes;   // forward, compensated (optional): [fwd_planes][ny][nx] partial sums
  float2* rtab;    // adjoint, compensated: [ny][npad] {cos, sin of the y-phase}
  float* ctab;     // adjoint, compensated: [nsx * kAdjCols][npad] x-phases
  float* partial;  // adjoint: [regions][npad][4]
  float* gpad;     // adjoint: G copied to a [ny][nsx*kAdjCols] zero-padded grid
  // separable variants
  float* sep_x;    // FP32: the contraction's x and y tables
  float* sep_y;
  float* sep_c;    // forward: partial planes [sep_splits][nyp][nxp]
  float4* fold;    // adjoint: partial sums [planes][npad]
  // half-precision separable variants: the contraction's tables and max |A|
  void *htab_x, *htab_y;
  unsigned* hmax;  // [kWave] maxima of |A|, as float bits
};

struct Plan {
  int64_t n, npad;
  int32_t nx, ny;
  int32_t variant, op;
  // forward
  int32_t fwd_gx, comp_gy, groups;
  bool comp_xtab;  // the compensated forward has its column table
  bool comp_wide;  // that table would exceed kCompColTabMaxBytes
  int32_t f64_chunk, f64_slices;  // FP64 forward: points per chunk (0 slices: the direct kernel)
  int32_t fwd_planes;  // partial planes of the compensated forward (0: none of its own)
  int32_t rec_k;  // recurrence forward: consecutive pixels per lane
  // adjoint: runs of strip-rows per point group (regions = the most runs the
  // partial buffer holds; the launch may use fewer)
  int32_t nsx, regions, ngroups, adj_kind;
  int64_t strip_rows;
  AdjOrder adj_order;
  bool need_gpad;
  // separable variant
  int32_t nxp, nyp, sep_splits, sep_splits_u, sep_splits_p;
  int64_t k2, fold_planes;
  size_t off_sep_x, off_sep_y, off_sep_c, off_fold;
  size_t off_hx, off_hy, off_hmax;  // half variants
  size_t off_plain, off_amp, off_xrec, off_yrec, off_rec64, off_ytab, off_xtab, off_planes, off_tab64,
      off_planes64, off_rtab,
      off_ctab, off_partial, off_gpad, total;
};

// col_table = false plans the compensated forward without its column table
// (the kernel then forms the x-phases itself: the same bits, less scratch).
Plan make_plan(int64_t n, int32_t nx, int32_t ny, int32_t variant, int32_t op,
               bool col_table = true);
Workspace carve(const Plan& p, void* base);

// Launch wrappers (return the hipError_t of the launch).
hipError_t launch_prep(const float* x, const float* y, const float* z, const float* a, int64_t n,
                       int64_t npad, double pitch, double wavelength, const Workspace& w,
                       bool want64, hipStream_t s);
hipError_t launch_fill_zero_f32(float* p, int64_t count, hipStream_t s);
hipError_t launch_fill_zero_f64(double* p, int64_t count, hipStream_t s);
// The compensated forward's precompute: the point records (as launch_prep),
// the per-row y-phase table and (when planned) the column x-phase table, in
// one launch.
hipError_t launch_prep_ytab(const float* x, const float* y, const float* z, const float* a,
                            double pitch, double wavelength, const Plan& p, const Workspace& w,
                            hipStream_t s);
// The compensated adjoint's tables, from the FP32 inputs in one launch: for
// every row y_h and point j the cosine and sine of the compensated y-phase of
// y_h, and for every strip column x_h and point j the compensated x-phase of
// x_h.
hipError_t launch_prep_rtab(const float* x, const float* y, const float* z, const float* a,
                            double pitch, double wavelength, const Plan& p, const Workspace& w,
                            hipStream_t s);
hipError_t launch_residual(const float* hologram, const float* target, float* residual,
                           int64_t count, hipStream_t s);
// The plain and recurrence forwards, and residual = I - target with a target.
hipError_t launch_fwd_plain(const Plan& p, const float* x, const float* y, const float* z,
                            const float* a, double pitch, double wavelength, float* out,
                            const float* target, float* residual, hipStream_t s);
// With target and residual (both or neither) the compensated forward also
// writes residual = out - target in its store.
hipError_t launch_fwd_comp(const Plan& p, const Workspace& w, float* out, hipStream_t s,
                           const float* target = nullptr, float* residual = nullptr);
hipError_t launch_fwd_rec(const Plan& p, const float* x, const float* y, const float* z,
                          const float* a, double pitch, double wavelength, float* out,
                          const float* target, float* residual, hipStream_t s);
hipError_t launch_fwd_f64(const Plan& p, const Workspace& w, double* out, hipStream_t s);
hipError_t launch_pad_g(const Plan& p, const float* g, float* gpad, hipStream_t s);
// Operand formats of the matrix-core contractions (contract.h):
constexpr int kHalfF16 = 0;    // one fp16 plane per operand
constexpr int kHalfBF16 = 1;   // one bf16 plane per operand
constexpr int kHalfF16x3 = 2;  // fp16 hi + lo planes, hi*hi + hi*lo + lo*hi
constexpr int kF32 = 3;        // FP32

// Runs per point group for this launch (<= p.regions), from the occupancy of
// the adjoint kernel on the current device.
int adj_runs(const Plan& p);
hipError_t launch_adj_partial(const Plan& p, const Workspace& w, const float* x, const float* y,
                              const float* z, const float* a, double pitch, double wavelength,
                              const float* g, int64_t ldg, int runs, hipStream_t s);
hipError_t launch_adj_finalize(const Plan& p, const Workspace& w, const float* z, const float* a,
                               double pitch, double wavelength, int runs, float* gx, float* gy,
                               float* gz, float* ga, hipStream_t s);

}  // namespace cgh
