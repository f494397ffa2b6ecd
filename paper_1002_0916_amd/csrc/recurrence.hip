// Forward by the recurrence of Eq. (2) (Section 2.1): along a row the phase of
// pixel x_h + n follows from two additions, Gamma_n = Gamma_{n-1} + delta_{n-1}
// and delta_n = delta_{n-1} + Delta, from Gamma_0 = P r^2 at x_h, delta_0 = P (2
// (x_h - x_j) + 1) and Delta = 2 P (here in revolutions, P -> Prev).  Lane l
// covers the K consecutive pixels x0 + K l ... x0 + K l + K - 1 of R rows
// (the paper's work-item covers eight consecutive pixels of one row).  delta and
// Delta depend on the column only, so the lane's rows share them: per point the
// lane forms dx and delta_0 once and Gamma_0 = fract(Prev r^2) (the plain phase)
// once per row, and per interaction the recurrence costs one add for Gamma (and a
// quarter of one for delta) before the native cosine and the accumulate.
// Gamma_0 is in [0, 1) and delta_0, Delta are reduced mod 1 (exactly; cos is
// 1-periodic in revolutions), so |Gamma_n| < 1 + n (1 + n) stays well inside the
// cosine's exact-reduction range without a fract per step.
//
// The vector ALU bounds it: an add, the cosine and an fma are 3.7 clocks of a CU
// for 64 interactions when all operands are VGPRs and 4.0 when the amplitude is
// an SGPR, and the seeds add 0.6 at K = 8.  So the points {x, Prev, A, Delta} and the
// rows' y_h - y_j are staged in LDS per tile of kTile points and reach the lanes
// as broadcasts.  The eight waves of a workgroup share the pixels and take eight
// points of every tile each, since a lane's K x R pixels leave few waves (1024 of
// 64 K x 4 at 1920x1024, for 8192 places); their sums are added in a fixed order.
// For many points on few pixels (order.h) the order of addition is that of two
// halves of the points, each in order.
// 1920x1080, N = 8192: 2345 us a call, where records in SGPRs and two groups of
// waves took 2671; 3840x2160, N = 1024: 1046 and 1166; 333x197, N = 700: 18 and 45.
#include <type_traits>

#include "cgh_internal.h"
#include "order.h"
#include "phase.h"

namespace cgh {

namespace {

constexpr int kWaves = 8;  // per workgroup

// A point's y_h - y_j at a lane's rows.
template <int R>
struct alignas(4 * R) Dy {
  float v[R];
};

// K pixels x R rows per lane; P parts of the points, each with kWaves / P waves on
// rows of their own.  Eight parts take eight points of every tile each; two take one
// half of all points each, in order.
template <int K, int R, int P>
__global__ __launch_bounds__(kWaves * kWave, 8) void fwd_rec_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int64_t n, int npad, double pitch, double wavelength, int nx,
    int ny, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  constexpr int kMine = kTile / P, kGroups = kWaves / P;
  __shared__ float4 recs[2][kTile];  // {x, Prev, A, Delta}
  __shared__ Dy<R> dys[2][kGroups][kTile];
  // The upper half of the parts leaves its sums for the lower half, and so on.
  __shared__ float sums[kWaves / 2 * R * K * kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int part = wave / kGroups, w = wave % kGroups;
  // (two dimensions, so that neither exceeds 2^32 threads on the largest holograms:
  // row blocks along x, up to 2^20, column blocks along y)
  const unsigned tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int x0 = ((int)(tile % gridDim.y) * kWave + lane) * K;
  const int y0 = ((int)(tile / gridDim.y) * kGroups + w) * R;
  const float xh = (float)x0;

  // The tile's stage: lane l has point l of it.  Every wave of part 0 forms its own
  // rows' dy, and the first one the records.
  float px = 0.0f, py = 0.0f, pz = 1.0f, pa = 0.0f;
  auto load = [&](int t) {
    const int64_t j = P == 2 ? (int64_t)(lane / kMine) * (npad / 2) + t * kMine + lane % kMine
                             : (int64_t)t * kTile + lane;
    const bool in = part == 0 && j < n, first = in && w == 0;
    py = in ? y[j] : 0.0f;
    px = first ? x[j] : 0.0f;
    pz = first ? z[j] : 1.0f;
    pa = first ? a[j] : 0.0f;
  };
  auto store = [&](int b) {
    if (part != 0) return;
    if (w == 0) {
      const float prev = (float)((pitch * pitch) / (2.0 * wavelength * (double)pz));
      recs[b][lane] = make_float4(px, prev, pa, fract(prev + prev));
    }
    Dy<R> dy;
#pragma unroll
    for (int i = 0; i < R; ++i) dy.v[i] = (float)(y0 + i) - py;
    dys[b][w][lane] = dy;
  };

  float acc[R][K];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int k = 0; k < K; ++k) acc[i][k] = 0.0f;
  const int ntiles = npad / kTile;
  load(0);
  store(0);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int b = t & 1;
    if (t + 1 < ntiles) load(t + 1);
#pragma unroll 2
    for (int q = 0; q < kMine; ++q) {
      const int p = part * kMine + q;
      const float4 r = recs[b][p];
      const Dy<R> dy = dys[b][w][p];
      const float dx = xh - r.x;
      const float dx2 = dx * dx;
      float d = fract(r.y * __builtin_fmaf(2.0f, dx, 1.0f));
      float g[R];
#pragma unroll
      for (int i = 0; i < R; ++i)
        g[i] = fract(r.y * __builtin_fmaf(dy.v[i], dy.v[i], dx2));
#pragma unroll
      for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i][k] = __builtin_fmaf(r.z, cos_rev(g[i]), acc[i][k]);
        if (k + 1 < K) {
#pragma unroll
          for (int i = 0; i < R; ++i) g[i] += d;
          d += r.w;
        }
      }
    }
    if (t + 1 < ntiles) store(b ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int left = P / 2; left >= 1; left /= 2) {
    float* at = sums + (part % left * kGroups + w) * R * K * kWave + lane;
    if (part >= left && part < 2 * left) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < K; ++k) at[(i * K + k) * kWave] = acc[i][k];
    }
    __syncthreads();
    if (part < left) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[i][k] += at[(i * K + k) * kWave];
    }
    __syncthreads();
  }
  if (part > 0) return;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (y0 + i >= ny) continue;
    const int64_t row = (int64_t)(y0 + i) * nx;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (x0 + k >= nx) continue;
      out[row + x0 + k] = acc[i][k];
      if (res) res[row + x0 + k] = acc[i][k] - tgt[row + x0 + k];
    }
  }
}

template <int K, int R, int P>
hipError_t launch(const Plan& p, const float* x, const float* y, const float* z, const float* a,
                  double pitch, double wavelength, float* out, const float* target,
                  float* residual, hipStream_t s) {
  const int64_t tiles_x = ((int64_t)p.nx + kWave * K - 1) / (kWave * K);
  constexpr int kRows = kWaves / P * R;
  const int64_t tiles_y = ((int64_t)p.ny + kRows - 1) / kRows;
  if (tiles_x * tiles_y > 0x7fffffff || tiles_x > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL((fwd_rec_kernel<K, R, P>), dim3((unsigned)tiles_y, (unsigned)tiles_x),
                     dim3(kWaves * kWave), 0, s, x, y, z, a, p.n, (int)p.npad, pitch, wavelength,
                     p.nx, p.ny, out, target, residual);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_rec(const Plan& p, const float* x, const float* y, const float* z,
                          const float* a, double pitch, double wavelength, float* out,
                          const float* target, float* residual, hipStream_t s) {
  auto go = [&](auto f) { return f(p, x, y, z, a, pitch, wavelength, out, target, residual, s); };
  auto shape = [&](auto k) {
    constexpr int K = decltype(k)::value;
    // Many points on few pixels: two sums of half the points each, in order.  Its
    // workgroups run in rounds of 256, one a CU, and a round of 2 rows per lane takes
    // 1.7 times one of 1 row, 4 rows as long as two of 2.  (us at 1 and 2 rows:
    // 365x339, N = 10048: 469 and 764; 213x1332, N = 14185: 1166 and 1084; 1065x967, N
    // = 51492: 8642 and 10371; 1786x835, N = 65536: 14832 and 13446.)
    if (ordered_sum(p.n, p.nx, p.ny)) {
      const int64_t cols = ((int64_t)p.nx + kWave * K - 1) / (kWave * K);
      const int64_t one = (cols * (((int64_t)p.ny + 3) / 4) + 255) / 256;
      const int64_t two = (cols * (((int64_t)p.ny + 7) / 8) + 255) / 256;
      return 10 * one < 17 * two ? go(launch<K, 1, 2>) : go(launch<K, 2, 2>);
    }
    // Waves of 64 K x 4 pixels: few of them take fewer rows per lane, so that there
    // are more waves, at more seeds per pixel.  (us at 4, 2 and 1 rows: 160x245, N =
    // 2612: 107, 59, 40; 640x480, N = 512: 34, 33, 35; 1865x300, N = 2246: 238, 193,
    // 211; 1024x1024, N = 4096: 524, 570, 595.)
    const int64_t waves = ((int64_t)p.nx + kWave * K - 1) / (kWave * K) * (((int64_t)p.ny + 3) / 4);
    // (with so few K is 4)
    if constexpr (K == 4)
      if (waves <= 80) return go(launch<K, 1, 8>);
    if (waves <= 430) return go(launch<K, 2, 8>);
    return go(launch<K, 4, 8>);
  };
  if (p.rec_k == 4) return shape(std::integral_constant<int, 4>{});
  if (p.rec_k == 6) return shape(std::integral_constant<int, 6>{});
  return shape(std::integral_constant<int, 8>{});
}

}  // namespace cgh
