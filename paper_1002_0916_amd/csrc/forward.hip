// Direct forward kernels: the compensated sum of Eq. (1) (Section 1) of a few
// points and of many points on few pixels (order.h), and the FP64 one where the
// contraction's tables have no room.  The plain
// form is in plain.hip, Eq. (2) in recurrence.hip, the contractions in
// contract_fwd.hip and contract_f64.hip.
//
// Work mapping: one hologram column per lane.  The compensated kernel gives lane l
// of a wave column x0 + l and a few consecutive rows, so a wave writes fully
// coalesced 256-byte row segments; the FP64 one has one pixel per lane and reads
// the points through scalar loads.
#include "cgh_internal.h"
#include "phase.h"

namespace cgh {

namespace {

// Compensated FP32: the phase separates exactly as X_j(x_h) + Y_j(y_h) with
// X_j(x_h) = Prev (x_h - x_j)^2 and Y_j(y_h) = Prev (y_h - y_j)^2.  Each part
// is formed on the integer pixel grid as a compensated split product reduced
// mod 1 (axis_phase).  Lane l of a wave owns column col0 + l and the wave
// kCompRows rows; the kCompWaves waves of a workgroup share their 64
// columns.  Per tile of kTile points the workgroup stages in LDS the x-phases
// [point][column] (from the column table xtab[col][npad] with TAB, else
// formed from each point's record: the same bits), each wave's row phases
// [point] (one float4 of the row table: its kCompRows rows) and the
// amplitudes.  The inner loop reads X per lane and Y and A as broadcast LDS
// reads (every lane the same address), so every operand of the per-
// interaction add, cosine and fma is a VGPR: on gfx950 such FP32 instructions
// issue about 1.7 times as fast as ones reading an SGPR, and without SGPR
// buffers the kernel fits eight waves per SIMD.  The tile is single-buffered
// (25 KB of LDS): the next tile's values are loaded into registers while the
// current one is consumed and stored between two barriers.  Per interaction:
// one add, the native cosine (no fract: the sum stays within a few
// revolutions) and one fma.
template <bool TAB, bool RES>
__device__ __forceinline__ void fwd_comp_body(const float* __restrict__ xrec,
                                                  const float* __restrict__ xtab,
                                                  const float* __restrict__ amp,
                                                  const float* __restrict__ ytab, int npad,
                                                  int nx, int ny, float* __restrict__ out,
                                                  const float* __restrict__ tgt,
                                                  float* __restrict__ res) {
  static_assert(kCompRows == 4, "a wave's row phases of one point are one float4");
  __shared__ float xs[kTile * kTilePitch];
  __shared__ float4 ys[kCompWaves][kTile];
  __shared__ float4 as4[kTile / 4];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // Tiles in column-major order, so each XCD takes a band of columns: it
  // reads only its columns' share of the column table (the larger table),
  // and all of the row table.
  const unsigned tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int by = (int)(tile % gridDim.y), bx = (int)(tile / gridDim.y);
  const int col = bx * kWave + lane;
  const int col0 = bx * kWave;
  const int grp = by * kCompWaves + wave;
  const float4* __restrict__ yt = reinterpret_cast<const float4*>(ytab) + (int64_t)grp * npad;
  const int ntiles = npad / kTile;
  constexpr int kColsPerWave = kWave / kCompWaves;
  const __amdgpu_buffer_rsrc_t xtab_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(xtab), 0, TAB ? (int)((int64_t)gridDim.x * kWave * npad * 4) : 0,
      0x00020000);

  // Registers holding the next tile: lane l of wave w has point l's x-phases
  // of the wave's kColsPerWave columns (or its record), its row phases, and
  // (wave 0) its amplitude.
  float xv[kColsPerWave];
  float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), yv;
  float r1 = 0.f, av = 0.f;
  auto load_tile = [&](int t) {
    const int j = t * kTile + lane;
    if (TAB) {
#pragma unroll
      for (int k = 0; k < kColsPerWave; ++k) {
        const int c = col0 + wave * kColsPerWave + k;
        xv[k] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(
                       xtab_rsrc, (unsigned)lane * 4u,
                       (int)(((int64_t)c * npad + (int64_t)t * kTile) * 4), 0));
      }
    } else {
      const float* r = xrec + (int64_t)j * kAxisRec;
      r0 = *reinterpret_cast<const float4*>(r);
      r1 = r[4];
    }
    yv = yt[j];
    if (wave == 0) av = amp[j];
  };
  auto store_tile = [&]() {
#pragma unroll
    for (int k = 0; k < kColsPerWave; ++k) {
      const int c = wave * kColsPerWave + k;
      xs[lane * kTilePitch + c] =
          TAB ? xv[k] : axis_phase((float)(col0 + c), r0.x, r0.y, r0.z, r0.w, r1);
    }
    ys[wave][lane] = yv;
    if (wave == 0) reinterpret_cast<float*>(as4)[lane] = av;
  };

  float acc[kCompRows];
#pragma unroll
  for (int i = 0; i < kCompRows; ++i) acc[i] = 0.0f;
  load_tile(0);
  priority_start();
  for (int t = 0; t < ntiles; ++t) {
    priority_step(t, ntiles);
    if (t > 0) __syncthreads();  // every wave is done with the previous tile
    store_tile();
    __syncthreads();
    if (t + 1 < ntiles) load_tile(t + 1);
#pragma unroll 2
    for (int p = 0; p < kTile; p += 8) {
#pragma unroll
      for (int q = 0; q < 8; q += 4) {
        const float4 a4 = as4[(p + q) / 4];
        const float A[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float X = xs[(p + q + u) * kTilePitch + lane];
          const float4 y4 = ys[wave][p + q + u];
          acc[0] = __builtin_fmaf(A[u], cos_rev(X + y4.x), acc[0]);
          acc[1] = __builtin_fmaf(A[u], cos_rev(X + y4.y), acc[1]);
          acc[2] = __builtin_fmaf(A[u], cos_rev(X + y4.z), acc[2]);
          acc[3] = __builtin_fmaf(A[u], cos_rev(X + y4.w), acc[3]);
        }
      }
    }
  }
  // The hologram, and in the RES instances the residual I - T (the upstream
  // gradient of 0.5 ||I - T||^2) in the same pass.  The two instances keep
  // the forward without a target at its own code: with the residual store
  // behind a run-time test, the same kernel ran about 1% slower at N >= 8192.
  const int y0 = grp * kCompRows;
  if (col < nx) {
#pragma unroll
    for (int i = 0; i < kCompRows; ++i) {
      if (y0 + i >= ny) continue;
      const int64_t idx = (int64_t)(y0 + i) * nx + col;
      out[idx] = acc[i];
      if constexpr (RES) res[idx] = acc[i] - tgt[idx];
    }
  }
}

__global__ __launch_bounds__(kCompThreads) void fwd_comp_kernel(
    const float* __restrict__ xtab, const float* __restrict__ amp, const float* __restrict__ ytab,
    int npad, int nx, int ny, float* __restrict__ out) {
  fwd_comp_body<true, false>(nullptr, xtab, amp, ytab, npad, nx, ny, out, nullptr, nullptr);
}

__global__ __launch_bounds__(kCompThreads) void fwd_comp_residual_kernel(
    const float* __restrict__ xtab, const float* __restrict__ amp, const float* __restrict__ ytab,
    int npad, int nx, int ny, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  fwd_comp_body<true, true>(nullptr, xtab, amp, ytab, npad, nx, ny, out, tgt, res);
}

__global__ __launch_bounds__(kCompThreads) void fwd_comp_inline_kernel(
    const float* __restrict__ xrec, const float* __restrict__ amp, const float* __restrict__ ytab,
    int npad, int nx, int ny, float* __restrict__ out) {
  fwd_comp_body<false, false>(xrec, nullptr, amp, ytab, npad, nx, ny, out, nullptr, nullptr);
}

__global__ __launch_bounds__(kCompThreads) void fwd_comp_inline_residual_kernel(
    const float* __restrict__ xrec, const float* __restrict__ amp, const float* __restrict__ ytab,
    int npad, int nx, int ny, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  fwd_comp_body<false, true>(xrec, nullptr, amp, ytab, npad, nx, ny, out, tgt, res);
}

// The residual G = I - T of an empty sum.
__global__ __launch_bounds__(256) void residual_kernel(const float* __restrict__ I,
                                                       const float* __restrict__ T,
                                                       float* __restrict__ G, int64_t count) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) G[t] = I[t] - T[t];
}

// FP64 reference: rho = Prev ((x_h - x_j)^2 + (y_h - y_j)^2) in revolutions,
// reduced exactly by rint, cosine by the device cospi.  One pixel per lane.
__global__ __launch_bounds__(256) void fwd_f64_kernel(const double4* __restrict__ rec, int npad,
                                                      int nx, int64_t npix,
                                                      double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npix) return;
  const double xh = (double)(p % nx);
  const double yh = (double)(p / nx);
  double acc = 0.0;
  for (int j = 0; j < npad; ++j) {
    const double4 r = rec[j];
    const double dx = xh - r.x;
    const double dy = yh - r.y;
    const double rho = r.z * (dx * dx + dy * dy);
    const double f = rho - rint(rho);
    acc += r.w * cospi(2.0 * f);
  }
  out[p] = acc;
}

}  // namespace

hipError_t launch_fwd_comp(const Plan& p, const Workspace& w, float* out, hipStream_t s,
                           const float* target, float* residual) {
  if ((target == nullptr) != (residual == nullptr)) return hipErrorInvalidValue;
  const dim3 grid(p.fwd_gx, p.comp_gy), block(kCompThreads);
  const float *xtab = w.xtab, *xrec = w.xrec, *amp = w.amp, *ytab = w.ytab;
  const int npad = (int)p.npad;
  if (w.xtab && residual)
    hipLaunchKernelGGL(fwd_comp_residual_kernel, grid, block, 0, s, xtab, amp, ytab, npad, p.nx,
                       p.ny, out, target, residual);
  else if (w.xtab)
    hipLaunchKernelGGL(fwd_comp_kernel, grid, block, 0, s, xtab, amp, ytab, npad, p.nx, p.ny,
                       out);
  else if (residual)
    hipLaunchKernelGGL(fwd_comp_inline_residual_kernel, grid, block, 0, s, xrec, amp, ytab, npad,
                       p.nx, p.ny, out, target, residual);
  else
    hipLaunchKernelGGL(fwd_comp_inline_kernel, grid, block, 0, s, xrec, amp, ytab, npad, p.nx,
                       p.ny, out);
  return hipGetLastError();
}

hipError_t launch_residual(const float* hologram, const float* target, float* residual,
                           int64_t count, hipStream_t s) {
  const unsigned blocks = grid_blocks(count, 256);
  if (!blocks) return hipErrorInvalidValue;
  hipLaunchKernelGGL(residual_kernel, dim3(blocks), dim3(256), 0, s, hologram, target, residual,
                     count);
  return hipGetLastError();
}

hipError_t launch_fwd_f64(const Plan& p, const Workspace& w, double* out, hipStream_t s) {
  const int64_t npix = (int64_t)p.nx * p.ny;
  const unsigned blocks = grid_blocks(npix, 256);
  if (!blocks) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fwd_f64_kernel, dim3(blocks), dim3(256), 0, s,
                     (const double4*)w.rec64, (int)p.npad, p.nx, npix, out);
  return hipGetLastError();
}

}  // namespace cgh
