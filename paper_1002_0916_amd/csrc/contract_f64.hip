// FP64 reference hologram as a contraction on the FP64 matrix cores.
//
// With X_j(x) = Prev (x_h - x_j)^2 and Y_j(y) = Prev (y_h - y_j)^2 in FP64
// revolutions, each reduced exactly by rint before its cosine and sine,
//
//   I[y][x] = sum_j A_j (cY_j(y) cX_j(x) - sY_j(y) sX_j(x))     (Eq. (1), Section 1)
//
// is a contraction of per-axis tables: two FP64 multiply-adds per point and
// pixel instead of a reduction and a cosine (about 60 FP64 instructions: 2.84 ms
// at 1920x1024, N = 1024).  The points are taken in chunks whose tables fit
// kF64TableBytes; later chunks add to the hologram.
//
// v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and
// accumulator r of lane l is D[4 r + l / 16][l % 16] (checked on the device).
// A wave computes 64 x 64 pixels (4 x 4 blocks: 16 MFMAs of 64 cycles for 8
// operand values, so the operands come straight from the tables), the four
// waves of a workgroup share the tile and split the points, and their sums are
// added in wave order through LDS (a fixed order: bitwise reproducible).  A
// table holds, per quad of points and coordinate, four pairs of doubles: pair q
// is what lanes l / 16 = q take in two successive MFMAs, (c0, c2), (s0, s2),
// (c1, c3), (s1, s3) of the quad's points, so a wave's load is 1 KB of
// consecutive bytes.
#include "contract.h"
#include "records.h"

namespace cgh {

namespace {

typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kF64Tile = 64;
constexpr int kF64Waves = 4;
constexpr int kF64Band = 8;        // tile rows per band of the tile order
constexpr int kF64TabRows = 64;    // coordinates per table workgroup

// One term of the sum, as the direct form has it.
__device__ __forceinline__ double term64(const double4& r, double x, double y) {
  const double dx = x - r.x, dy = y - r.y;
  const double rho = r.z * (dx * dx + dy * dy);
  return r.w * cospi(2.0 * (rho - rint(rho)));
}

// Stores pixel (row, col): the first chunk's sum, or the hologram plus it.  A
// sum that is not finite at the last chunk (an infinite or NaN amplitude or
// record, or an overflow) is taken again term by term, so that infinities and
// NaNs are the direct sum's.
__device__ __forceinline__ void finish64(double v, int64_t row, int64_t col, int nx, bool add,
                                         bool last, const double4* __restrict__ rec, int64_t n,
                                         double* __restrict__ out) {
  const int64_t idx = row * nx + col;
  if (add) v += out[idx];
  if (last && !(fabs(v) < __builtin_inf())) {
    v = 0.0;
    for (int64_t j = 0; j < n; ++j) v += term64(rec[j], (double)col, (double)row);
  }
  out[idx] = v;
}

// points [0, points) of the chunk in slices of per_slice (multiples of 16); with
// planes, slice s stores its raw sums to plane s.
__global__ __launch_bounds__(kWave* kF64Waves, 1) void contract_f64_kernel(
    const doublex2* __restrict__ yq, const doublex2* __restrict__ xq, int points, int per_slice,
    int rows, int cols, int nx, int ny, unsigned tiles_x, unsigned tiles, double* __restrict__ out,
    double* __restrict__ planes, bool add, bool last, const double4* __restrict__ rec,
    int64_t n) {
  constexpr int kB = kF64Tile / 16;      // blocks per side
  constexpr int kRegs = kB * kB * 4;     // accumulators per lane
  constexpr int kRounds = 2;             // of the final sums, 64 KB each
  constexpr int kChunk = kRegs / kRounds, kOwn = kChunk / kF64Waves;
  __shared__ doublex2 lds[kF64Waves * kChunk * kWave / 2];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int l16 = lane & 15, q = lane >> 4;
  const unsigned id = xcd_tile(blockIdx.x, gridDim.x);
  const unsigned slice = id / tiles, tile = id - slice * tiles;
  const unsigned band = tile / (kF64Band * tiles_x), in_band = tile - band * kF64Band * tiles_x;
  const unsigned bh = min((unsigned)kF64Band, tiles / tiles_x - band * kF64Band);
  const int x0 = (int)(in_band / bh) * kF64Tile;
  const int y0 = (int)(band * kF64Band + in_band % bh) * kF64Tile;

  // This wave's quads of points.
  const int first = (int)slice * per_slice;
  const int quads = (min(first + per_slice, points) - first) / 4 / kF64Waves;
  const int t0 = first / 4 + wave * quads, last_t = t0 + quads - 1;
  const doublex2* ybase = yq + (size_t)t0 * rows * 4 + (size_t)(y0 + l16) * 4 + q;
  const doublex2* xbase = xq + (size_t)t0 * cols * 4 + (size_t)(x0 + l16) * 4 + q;
  doublex4 acc[kB][kB];
#pragma unroll
  for (int i = 0; i < kB; ++i)
#pragma unroll
    for (int k = 0; k < kB; ++k) acc[i][k] = doublex4{0.0, 0.0, 0.0, 0.0};
  doublex2 a[kB], b[kB];
#pragma unroll
  for (int i = 0; i < kB; ++i) {
    a[i] = ybase[i * 64];
    b[i] = xbase[i * 64];
  }
  for (int t = t0; t <= last_t; ++t) {
    if (t < last_t) {
      ybase += (size_t)rows * 4;
      xbase += (size_t)cols * 4;
    }
    doublex2 an[kB], bn[kB];
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      an[i] = ybase[i * 64];
      bn[i] = xbase[i * 64];
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < kB; ++i)
#pragma unroll
        for (int k = 0; k < kB; ++k)
          acc[i][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][e], b[k][e], acc[i][k], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      a[i] = an[i];
      b[i] = bn[i];
    }
  }

  double* sums = reinterpret_cast<double*>(lds);
#pragma unroll
  for (int h = 0; h < kRounds; ++h) {
    if (h > 0) __syncthreads();
#pragma unroll
    for (int c = 0; c < kChunk; c += 2) {
      const int r = h * kChunk + c;
      lds[((wave * kChunk + c) / 2) * kWave + lane] =
          doublex2{acc[r / 4 / kB][r / 4 % kB][r % 4], acc[r / 4 / kB][r / 4 % kB][r % 4 + 1]};
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kOwn; ++c) {
      const int r = h * kChunk + wave * kOwn + c;
      const int row = y0 + r / 4 / kB * 16 + 4 * (r % 4) + q;
      const int col = x0 + r / 4 % kB * 16 + l16;
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < kF64Waves; ++k) {
        const int at = k * kChunk + wave * kOwn + c;
        v += sums[((at / 2) * kWave + lane) * 2 + (at & 1)];
      }
      if (row < ny && col < nx) {
        if (planes)
          planes[((int64_t)slice * ny + row) * nx + col] = v;
        else
          finish64(v, row, col, nx, add, last, rec, n, out);
      }
    }
  }
}

// out (+)= the sum of the slices' planes, in slice order.
__global__ __launch_bounds__(256) void contract_f64_sum_kernel(
    const double* __restrict__ planes, int slices, int nx, int64_t count,
    double* __restrict__ out, bool add, bool last, const double4* __restrict__ rec, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  double v = 0.0;
#pragma unroll 8
  for (int k = 0; k < slices; ++k) v += planes[k * count + i];
  finish64(v, i / nx, i % nx, nx, add, last, rec, n, out);
}

// Tables of the chunk's points [j0, j0 + points): a workgroup is 16 points and
// kF64TabRows coordinates (y slices, then x slices).  Lane l of wave w takes
// point 4 w + l % 4 and coordinates l / 4, l / 4 + 16, ...  The first slice also
// writes the points' records.
__global__ __launch_bounds__(256) void contract_f64_tables_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int64_t n, int64_t j0, double pitch, double wavelength,
    int yslices, int rows, int cols, double* __restrict__ yq, double* __restrict__ xq,
    double4* __restrict__ rec) {
  const int lane = threadIdx.x & 63, e = lane & 3;
  const int64_t quad = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t j = j0 + quad * 4 + e;
  const bool is_y = (int)blockIdx.y < yslices;
  const int slice = is_y ? (int)blockIdx.y : (int)blockIdx.y - yslices;
  const PointRecord r = point_record(x, y, z, a, j, n, pitch, wavelength);
  if (blockIdx.y == 0 && lane < 4)
    rec[j] = make_double4((double)r.x, (double)r.y, r.prev, (double)r.a);
  const double at = (double)(is_y ? r.y : r.x), A = is_y ? (double)r.a : 1.0;
  const int size = is_y ? rows : cols;
  // pair of the cosine: 0 for points 0 and 2 of the quad, 2 for 1 and 3; the
  // sine's is the next one; the point's half of the quad is the place in a pair
  double* dst = (is_y ? yq : xq) + (quad * size) * 8 + (e & 1) * 4 + (e >> 1);
  for (int i = 0; i < kF64TabRows / 16; ++i) {
    const int h = slice * kF64TabRows + (lane >> 2) + 16 * i;
    const double d = (double)h - at, rho = r.prev * (d * d);
    double s, c;
    sincospi(2.0 * (rho - rint(rho)), &s, &c);
    dst[(int64_t)h * 8] = A * c;
    dst[(int64_t)h * 8 + 2] = is_y ? -(A * s) : s;
  }
}

inline int64_t round64(int64_t v) { return (v + 63) / 64 * 64; }

}  // namespace

void plan_contract_f64(Plan& p) {
  const int64_t rows = round64(p.ny), cols = round64(p.nx);
  const int64_t fit = kF64TableBytes / (16 * (rows + cols)) / 64 * 64;
  p.f64_chunk = (int32_t)std::min(p.npad, fit);
  p.f64_slices = 0;
  if (p.f64_chunk < 64) return;  // not even 64 points' tables fit
  // Fewer tiles than CUs: the chunk's points in slices, of 128 points at least.
  const int64_t tiles = rows / kF64Tile * (cols / kF64Tile);
  int64_t s = std::max<int64_t>(1, std::min<int64_t>(256 / tiles, p.f64_chunk / 128));
  const int64_t per = (p.f64_chunk / 64 + s - 1) / s;
  p.f64_slices = (int32_t)((p.f64_chunk / 64 + per - 1) / per);
}

size_t contract_f64_table_bytes(const Plan& p) {
  return (size_t)p.f64_chunk * 16 * (size_t)(round64(p.ny) + round64(p.nx));
}

hipError_t launch_contract_f64(const Plan& p, const Workspace& w, const float* x, const float* y,
                               const float* z, const float* a, double pitch, double wavelength,
                               double* out, hipStream_t s) {
  const int rows = (int)round64(p.ny), cols = (int)round64(p.nx);
  const unsigned tiles_x = cols / kF64Tile;
  const int64_t tiles = (int64_t)tiles_x * (rows / kF64Tile);
  if (tiles * p.f64_slices > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t pixels = (int64_t)p.nx * p.ny;
  double* yq = w.tab64;
  double* xq = yq + (size_t)p.f64_chunk * rows * 2;
  const int yslices = rows / kF64TabRows, xslices = cols / kF64TabRows;
  for (int64_t j0 = 0; j0 < p.npad; j0 += p.f64_chunk) {
    const int points = (int)std::min<int64_t>(p.f64_chunk, p.npad - j0);
    const bool add = j0 > 0, last = j0 + points == p.npad;
    hipLaunchKernelGGL(contract_f64_tables_kernel,
                       dim3((unsigned)(points / 16), (unsigned)(yslices + xslices)), dim3(256), 0,
                       s, x, y, z, a, p.n, j0, pitch, wavelength, yslices, rows, cols, yq, xq,
                       w.rec64);
    const int units = points / 64;
    const int per = (units + p.f64_slices - 1) / p.f64_slices;
    const int slices = (units + per - 1) / per;
    double* planes = slices > 1 ? w.planes64 : nullptr;
    hipLaunchKernelGGL(contract_f64_kernel, dim3((unsigned)(tiles * slices)),
                       dim3(kWave * kF64Waves), 0, s, (const doublex2*)yq, (const doublex2*)xq,
                       points, per * 64, rows, cols, p.nx, p.ny, tiles_x, (unsigned)tiles, out,
                       planes, add, last, w.rec64, p.n);
    if (planes)
      hipLaunchKernelGGL(contract_f64_sum_kernel, dim3(grid_blocks(pixels, 256)), dim3(256), 0, s,
                         planes, slices, p.nx, pixels, out, add, last, w.rec64, p.n);
  }
  return hipGetLastError();
}

}  // namespace cgh
