// Forward of the plain FP32 phase (Eq. (1), Section 1): per interaction the
// phase Prev ((x_h - x_j)^2 + (y_h - y_j)^2) in revolutions, reduced mod 1, the
// native cosine, and one fma.
//
// The kernel is bound by the vector ALU, where an FP32 instruction of VGPRs
// alone issues in 0.6 to 0.7 clocks of a CU, one that reads an SGPR or takes a
// fract in 1.1, and the cosine in 2.1.  So the points' values reach the lanes as
// LDS broadcasts, not as SGPRs: lane l of a wave has column x0 + l and R
// rows, and reads of each point {x, Prev, A} and its rows' y_h - y_j, which the
// workgroup forms once per tile of kTile points.  The fract is left out where it
// changes nothing: the cosine reduces up to 256 revolutions exactly, and each
// wave bounds the phase of every point of a tile over its own pixels.  That
// leaves an fma, a product, the cosine and an fma, 4.1 clocks, and 0.2 for dx^2.
// Several groups of waves share the pixels and split the points, so that small
// holograms fill the SIMDs too, but for many points on few pixels (order.h), where
// one group adds them all in order.  1920x1024, N = 1024: 281 us a call, where 8 rows
// per lane with the points in SGPRs took 384; 333x197, N = 700: 19 and 124.
#include <type_traits>

#include "cgh_internal.h"
#include "order.h"
#include "phase.h"

namespace cgh {

namespace {

constexpr int kPlainWaves = 8;         // per workgroup
constexpr float kExactCos = 255.0f;    // revolutions

// R rows per lane; S groups of kPlainWaves / S waves share the pixels and split
// the points.
template <int R, int S>
__global__ __launch_bounds__(kPlainWaves * kWave) void fwd_plain_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int64_t n, int npad, double pitch, double wavelength, int nx,
    int ny, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  constexpr int kQuads = R / 4, kGroup = kPlainWaves / S;
  __shared__ float4 recs[2][kTile];                         // {x, y, Prev, A}
  __shared__ float4 dys[2][kGroup][kTile][kQuads];
  __shared__ float sums[S > 1 ? (S - 1) * R * kGroup * kWave : 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int part = wave / kGroup, w = wave % kGroup;
  // (two dimensions, so that neither exceeds 2^32 threads on the largest holograms)
  const unsigned tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int x0 = (int)(tile % gridDim.x) * kWave, col = x0 + lane;
  const int y0 = ((int)(tile / gridDim.x) * kGroup + w) * R;
  const float xh = (float)col;

  // The tile's stage: lane l has point l.  Every wave of part 0 forms its own
  // rows' dy, and the first wave the records.
  float px = 0.0f, py = 0.0f, pz = 1.0f, pa = 0.0f;
  auto load = [&](int t) {
    const int64_t j = (int64_t)t * kTile + lane;
    px = py = pa = 0.0f;
    pz = 1.0f;
    if (j < n) {
      py = y[j];
      if (w == 0) {
        px = x[j];
        pz = z[j];
        pa = a[j];
      }
    }
  };
  auto store = [&](int b) {
    if (part != 0) return;
    if (w == 0)
      recs[b][lane] = make_float4(
          px, py, (float)((pitch * pitch) / (2.0 * wavelength * (double)pz)), pa);
#pragma unroll
    for (int q = 0; q < kQuads; ++q)
      dys[b][w][lane][q] =
          make_float4((float)(y0 + 4 * q) - py, (float)(y0 + 4 * q + 1) - py,
                      (float)(y0 + 4 * q + 2) - py, (float)(y0 + 4 * q + 3) - py);
  };

  float acc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) acc[i] = 0.0f;
  const int ntiles = npad / kTile;
  constexpr int kMine = kTile / S;
  load(0);
  store(0);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int b = t & 1;
    if (t + 1 < ntiles) load(t + 1);
    // The largest phase of point `lane` over the wave's pixels.
    const float4 mine = recs[b][lane];
    const float dxm = fmaxf(fabsf((float)x0 - mine.x), fabsf((float)(x0 + kWave - 1) - mine.x));
    const float dym =
        fmaxf(fabsf((float)y0 - mine.y), fabsf((float)(y0 + R - 1) - mine.y));
    const bool exact = fabsf(mine.z) * (dxm * dxm + dym * dym) <= kExactCos;
    auto points = [&](auto reduce) {
#pragma unroll 4
      for (int k = 0; k < kMine; ++k) {
        const int p = part * kMine + k;
        const float4 r = recs[b][p];
        const float dx = xh - r.x;
        const float dx2 = dx * dx;
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
          const float4 d = dys[b][w][p][q];
          const float dy[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = r.z * __builtin_fmaf(dy[i], dy[i], dx2);
            acc[4 * q + i] =
                __builtin_fmaf(r.w, cos_rev(decltype(reduce)::value ? fract(v) : v), acc[4 * q + i]);
          }
        }
      }
    };
    constexpr unsigned long long kAll = ~0ull >> (kTile - kMine);
    if (((__ballot(exact) >> (part * kMine)) & kAll) == kAll)
      points(std::false_type{});
    else
      points(std::true_type{});
    if (t + 1 < ntiles) store(b ^ 1);
    __syncthreads();
  }
  if constexpr (S > 1) {
    float* d = sums + w * R * kWave + lane;
    constexpr int kPart = kGroup * R * kWave;
    if (part > 0) {
#pragma unroll
      for (int i = 0; i < R; ++i) d[(part - 1) * kPart + i * kWave] = acc[i];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int q = 0; q < S - 1; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i) acc[i] += d[q * kPart + i * kWave];
  }
  if (col < nx) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (y0 + i >= ny) continue;
      const int64_t at = (int64_t)(y0 + i) * nx + col;
      out[at] = acc[i];
      if (res) res[at] = acc[i] - tgt[at];
    }
  }
}

template <int R, int S>
hipError_t launch(const Plan& p, const float* x, const float* y, const float* z, const float* a,
                  double pitch, double wavelength, float* out, const float* target,
                  float* residual, hipStream_t s) {
  constexpr int kRows = kPlainWaves / S * R;
  const int64_t tiles_x = (p.nx + kWave - 1) / kWave;
  const int64_t tiles_y = ((int64_t)p.ny + kRows - 1) / kRows;
  if (tiles_x * tiles_y > 0x7fffffff || tiles_y > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL((fwd_plain_kernel<R, S>), dim3((unsigned)tiles_x, (unsigned)tiles_y),
                     dim3(kPlainWaves * kWave), 0, s, x, y, z, a, p.n, (int)p.npad, pitch,
                     wavelength, p.nx, p.ny, out, target, residual);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_plain(const Plan& p, const float* x, const float* y, const float* z,
                            const float* a, double pitch, double wavelength, float* out,
                            const float* target, float* residual, hipStream_t s) {
  auto go = [&](auto f) { return f(p, x, y, z, a, pitch, wavelength, out, target, residual, s); };
  // Many points on few pixels: all of them in one sum, in order.
  if (ordered_sum(p.n, p.nx, p.ny)) return go(launch<4, 1>);
  // Waves of 64 x 4 pixels, of which the chip holds 8192: few of them split the
  // points further, and many let a lane keep 8 rows, which share a point's dx^2
  // and reads.  (us at 4 rows and 8 parts, 4 and 4, 8 and 2: 640x480, N = 512:
  // 29, 32, 46; 1865x300, N = 2246: 215, 229, 365; 331x1665, N = 7102: 694, 662,
  // 1029; 1920x1024, N = 1024: 314, 305, 346; 3840x2160, N = 1024: 1352, 1286,
  // 1185.)
  const int64_t waves = ((int64_t)p.nx + kWave - 1) / kWave * (((int64_t)p.ny + 3) / 4);
  if (waves <= 2300) return go(launch<4, 8>);
  if (waves <= 16384) return go(launch<4, 4>);
  return go(launch<8, 2>);
}

}  // namespace cgh
