// Forward hologram as one contraction on the matrix cores (contract.h):
//
//   I[y][x] = sum_j A_j (cY_j(y) cX_j(x) - sY_j(y) sX_j(x)) = sum_k P[y][k] Q[x][k],
//   P[y][2j] = A_j cY_j(y), P[y][2j + 1] = -A_j sY_j(y), Q[x][2j] = cX_j(x),
//   Q[x][2j + 1] = sX_j(x)                                      (Eq. (1), Section 1)
//
// A wave computes MI x NJ blocks of 32 x 32 pixels with
// v_mfma_f32_32x32x16 (lane l: row or column l % 32, k = (l / 32) * 8 .. + 7,
// i.e. four points; accumulator register r: row (r / 4) * 8 + (l / 32) * 4 +
// r % 4, column l % 32).  The operands never exist in memory: a lane reads the
// phases of its four points at its coordinate (16 bytes), takes their cosines
// and sines and splits them into fp16 planes in registers, already in the
// matrix cores' layout.  The table is therefore 4 bytes per point and
// coordinate where both planes of both values would be 8.
//
// A workgroup is KS groups of WM waves.  The WM waves of a group are stacked in
// y and share their columns: each forms a share of the column operand and
// leaves it in LDS (double buffered), in the layout in which all of them read
// it back (a wave reads or writes 1 KB of consecutive bytes: no bank
// conflicts).  The row operand stays in the registers of the wave that forms
// it.  The KS groups split the points of the same pixels; their sums are added in
// group order through LDS at the end (a fixed order: bitwise reproducible), which
// also keeps every chain of additions short.
//
// With one group of one wave (KS = 1) a slice is one chain of additions in the order
// of its points.  The separable variants use it for many points on few pixels
// (order.h), with their plan's K splits as slices, so that a sum is the same however
// the other shapes cut it: the operands are then without the factor 1 + 2^-24, the
// f16x3 ones below 1, and FP32 pairs point p of 16 with point p + 8.
//
// The FP32 format (v_mfma_f32_32x32x2, 4 flops per interaction) is bound by the
// FP32 matrix cores, whose instructions occupy the vector unit as well: a cosine
// or sine beside them costs its full time, so its tables hold the operands
// themselves (8 bytes).  1920x1024, N = 1024: 88 us a call where a tiled product
// of operand tables in memory took 99 (333x197, N = 700: 16 and 32).
#include "contract.h"
#include "records.h"

namespace cgh {

namespace {

constexpr int kBand = 8;       // tile rows per band of the tile order
constexpr int kTabRows = 256;  // coordinates per table workgroup slice
constexpr int kAmaxInline = 8192;  // points up to which the tables find max |A| themselves

// (cos, sin) operand block share from four phases, times a factor each for the
// cosine and the sine.
template <int MODE>
__device__ __forceinline__ Frag frag_of_phases(float4 ph) {
  const float v[8] = {cos_rev(ph.x), sin_rev(ph.x), cos_rev(ph.y), sin_rev(ph.y),
                      cos_rev(ph.z), sin_rev(ph.z), cos_rev(ph.w), sin_rev(ph.w)};
  return make_frag<MODE>(v);
}
template <int MODE, bool RAISE = true>
__device__ __forceinline__ Frag frag_of_phases(float4 ph, float4 a) {
  const float v[8] = {a.x * cos_rev(ph.x), -(a.x * sin_rev(ph.x)), a.y * cos_rev(ph.y),
                      -(a.y * sin_rev(ph.y)), a.z * cos_rev(ph.z), -(a.z * sin_rev(ph.z)),
                      a.w * cos_rev(ph.w), -(a.w * sin_rev(ph.w))};
  return make_frag<MODE, RAISE>(v);
}

// One quad's phases at coordinate h from its records {c, ph, pl, b, d}.
__device__ __forceinline__ float4 quad_phases(const float4* __restrict__ rec, int64_t q, float h) {
  const float4 c = rec[q * 5], ph = rec[q * 5 + 1], pl = rec[q * 5 + 2], b = rec[q * 5 + 3],
               d = rec[q * 5 + 4];
  return make_float4(axis_phase(h, c.x, ph.x, pl.x, b.x, d.x),
                     axis_phase(h, c.y, ph.y, pl.y, b.y, d.y),
                     axis_phase(h, c.z, ph.z, pl.z, b.z, d.z),
                     axis_phase(h, c.w, ph.w, pl.w, b.w, d.w));
}

template <int MODE, int MI, int NJ, int WM, int KS, bool XTAB, bool RES>
__global__ __launch_bounds__(kWave* WM* KS, 2) void contract_fwd_kernel(
    FwdOperands o, int npad, int nx, int ny, unsigned tiles_x, unsigned tiles, int per_slice,
    const unsigned* __restrict__ amax, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  constexpr bool kForms = MODE == kHalfF16x3;  // from phases; else the tables hold operands
  constexpr bool kInOrder = KS == 1;
  constexpr int kFar = kInOrder && MODE == kF32 ? 2 : 1;  // quads between the lanes' halves
  constexpr int kThreads = kWave * WM * KS;
  constexpr int kPlanes = kForms || MODE == kF32 ? 2 : 1;  // uint4 per operand share
  constexpr int kLoad = MODE == kF32 ? 2 : 1;              // and per table entry
  constexpr int kS = 2;                          // steps (of 8 points) per LDS stage
  constexpr int kShare = WM > 1 ? kS * NJ / WM : 1;  // operand blocks a wave forms per stage
  constexpr int kAhead = 2;                      // steps whose phases are loaded ahead
  constexpr int kPx = WM > 1 ? kShare : NJ;
  static_assert(WM == 1 || kS * NJ % WM == 0, "the waves of a group share a stage evenly");
  constexpr int kStage = WM > 1 ? 2 * kS * NJ * kPlanes * kWave : 0;  // uint4 per group
  constexpr int kRegs = MI * NJ * 16;               // accumulators per lane
  constexpr int kRounds = (KS * WM * kRegs + 255) / 256;  // of the final sums, 64 KB each
  constexpr int kChunk = kRegs / kRounds;           // registers per wave and round
  constexpr int kOwn = kChunk / KS;                 // of these, summed by one group
  constexpr int kVec = kOwn < 4 ? kOwn : 4;
  static_assert(kOwn >= 1 && kOwn * KS * kRounds == kRegs, "the groups share every round evenly");
  constexpr int kSum = KS * WM * kChunk * kWave / 4;
  constexpr int kLds = KS * kStage > kSum ? KS * kStage : kSum;
  __shared__ uint4 lds[kLds];
  __shared__ unsigned red[WM * KS];

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int grp = wave / WM, w = wave % WM;
  const int half = lane >> 5, l32 = lane & 31;
  // Slices of the points in order, each with all tiles; slice s writes (or is)
  // plane s of the output.
  const unsigned id = xcd_tile(blockIdx.x, gridDim.x);
  const unsigned slice = id / tiles, tile = id - slice * tiles;
  out += (int64_t)slice * nx * ny;
  // Bands of kBand tile rows, each walked column by column: the tiles that run
  // together on an XCD are then about square and share both tables' parts.
  const unsigned band = tile / (kBand * tiles_x), in_band = tile - band * kBand * tiles_x;
  const unsigned bh = min((unsigned)kBand, tiles / tiles_x - band * kBand);
  const int tx = (int)(in_band / bh), ty = (int)(band * kBand + in_band % bh);
  const int y0 = ty * (WM * MI * 32) + w * (MI * 32), x0 = tx * (NJ * 32);

  // Step t: points 8 t .. 8 t + 7, quads 2 t + half.  Rows and columns beyond
  // the tables repeat the last one (their pixels are not stored).
  const int first = (int)slice * per_slice;  // points, multiples of 64
  const int steps = (min(first + per_slice, npad) - first) / 8 / KS;
  const int t0 = first / 8 + grp * steps;
  const int last = t0 + steps - 1;
  const char* __restrict__ yt = static_cast<const char*>(o.yq);
  const char* __restrict__ xt = static_cast<const char*>(o.xq);
  const char* __restrict__ at = reinterpret_cast<const char*>(o.amp);
  // This lane's byte offsets within a step (uniform base + 32-bit offset).
  unsigned yoff[MI], xoff[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
    yoff[i] = (unsigned)(half * kFar * o.rows_y + min(y0 + i * 32 + l32, o.rows_y - 1)) * 16u;
#pragma unroll
  for (int n = 0; n < NJ; ++n)
    xoff[n] = (unsigned)(half * kFar * o.cols_x + min(x0 + n * 32 + l32, o.cols_x - 1)) * 16u;
  // The first half's quad of step t.
  auto quad = [&](int t) -> int64_t {
    return kFar == 2 ? 4 * (int64_t)(t >> 1) + (t & 1) : 2 * (int64_t)t;
  };
  struct Entry {
    uint4 q[kLoad];
  };
  struct RowPhases {
    Entry p[MI];
    float4 a;
  };
  // kF32: a quad's second pair of points is a plane further.
  const int64_t yplane = (int64_t)(npad / 4) * o.rows_y * 16;
  const int64_t xplane = (int64_t)(npad / 4) * o.cols_x * 16;
  auto load_y = [&](int t, RowPhases& r) {
    const char* base = yt + quad(t) * o.rows_y * 16;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int k = 0; k < kLoad; ++k)
        r.p[i].q[k] = *reinterpret_cast<const uint4*>(base + k * yplane + yoff[i]);
    if (kForms) r.a = *reinterpret_cast<const float4*>(at + (int64_t)t * 32 + (unsigned)half * 16u);
  };
  auto load_x = [&](int t, int n) -> Entry {
    Entry p;
    if constexpr (XTAB) {
      const char* base = xt + quad(t) * o.cols_x * 16;
#pragma unroll
      for (int k = 0; k < kLoad; ++k)
        p.q[k] = *reinterpret_cast<const uint4*>(base + k * xplane + xoff[n]);
    } else {
      p.q[0] = __builtin_bit_cast(
          uint4, quad_phases(o.rec, (int64_t)t * 2 + half, (float)(x0 + n * 32 + l32)));
    }
    return p;
  };
  auto form_x = [&](const Entry& p) -> Frag {
    if constexpr (kForms) return frag_of_phases<MODE>(__builtin_bit_cast(float4, p.q[0]));
    return Frag{p.q[0], p.q[kLoad - 1]};
  };

  // The first kAhead steps' loads are in flight while the scale is found.
  RowPhases py[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) load_y(min(t0 + u, last), py[u]);
  Entry px[kPx];
  uint4* buf = lds + grp * kStage;
  constexpr int kBuf = kS * NJ * kPlanes * kWave;
  // WM > 1: this wave's share of stage s, blocks b = w, w + WM, ... of the
  // stage's kS * NJ (step b / NJ, column block b % NJ).
  auto load_block = [&](int s, int k) {
    const int b = k * WM + w;
    px[k] = load_x(min(t0 + s * kS + b / NJ, last), b % NJ);
  };
  auto store_block = [&](int s, int k) {
    const Frag f = form_x(px[k]);
    uint4* d = buf + (s & 1) * kBuf + (k * WM + w) * kPlanes * kWave + lane;
    d[0] = f.hi;
    if (kPlanes > 1) d[kWave] = f.lo;
  };
  auto load_stage = [&](int s) {
#pragma unroll
    for (int k = 0; k < kShare; ++k) load_block(s, k);
  };
  auto store_stage = [&](int s) {
#pragma unroll
    for (int k = 0; k < kShare; ++k) store_block(s, k);
  };
  if constexpr (WM == 1) {
#pragma unroll
    for (int n = 0; n < NJ; ++n) px[n] = load_x(t0, n);
  } else {
    load_stage(0);
  }

  // Scale of the amplitudes from their largest magnitude.
  unsigned m = 0;
  if (MODE == kHalfF16x3 && !kInOrder) {
    for (int j = threadIdx.x * 4; j < npad; j += kThreads * 4) {
      const float4 v = *reinterpret_cast<const float4*>(o.amp + j);
      m = max(m, max(max(__float_as_uint(fabsf(v.x)), __float_as_uint(fabsf(v.y))),
                     max(__float_as_uint(fabsf(v.z)), __float_as_uint(fabsf(v.w)))));
    }
    m = group_max<kThreads>(m, red);
  } else if (MODE != kF32) {
    m = group_max<kWave>(amax[lane], red);
  }
  float mul = 1.0f, undo = 1.0f;
  if (kInOrder && MODE != kF32)
    operand_scale<MODE, 0>(m, mul, undo);
  else if (MODE != kF32)
    operand_scale<MODE>(m, mul, undo);
  auto form_y = [&](const RowPhases& r, float mul, Frag (&A)[MI]) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if constexpr (kForms) {
        A[i] = frag_of_phases<MODE, !kInOrder>(
            __builtin_bit_cast(float4, r.p[i].q[0]),
            make_float4(r.a.x * mul, r.a.y * mul, r.a.z * mul, r.a.w * mul));
      } else {
        const uint4 zero = make_uint4(0, 0, 0, 0);
        A[i] = mul != 0.0f ? Frag{r.p[i].q[0], r.p[i].q[kLoad - 1]} : Frag{zero, zero};
      }
    }
  };

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int n = 0; n < NJ; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.0f;
  auto products = [&](const Frag (&A)[MI], const Frag& B, int n) {
    auto part = [&](auto k) {
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[i][n] = mfma_part<MODE, decltype(k)::value>(A[i], B, acc[i][n]);
    };
    parts(part, std::make_integer_sequence<int, mfmas_per_step(MODE)>{});
  };

  // The matrix cores run beside the vector ALU only if a wave keeps issuing
  // vector instructions between its MFMAs, so the operands of the next step are
  // formed among the products of the current one, in the proportion given here.
  // (On gfx950 the same instructions as two blocks take 1.5 times as long.)
  constexpr int kForm = MI + (WM == 1 ? NJ : kShare / kS);  // quads formed per step
  constexpr int kMfma = MI * NJ * mfmas_per_step(MODE);     // MFMAs per step
  auto interleave = [&]() {
    if constexpr (kForms) {
      constexpr int kTrans = (kForm * 8 + kMfma - 1) / kMfma;
      constexpr int kValu = (kForm * 16 + kMfma - 1) / kMfma;
#pragma unroll
      for (int k = 0; k < kMfma; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, kTrans, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
      }
    }
  };
  Frag A[2][MI];
  if constexpr (WM == 1) {
    // Column block n + 1 (or the next step's first) is formed among block n's
    // products, and the next step's rows among all of them.  An odd last step
    // is taken with zero amplitudes.
    Frag B = form_x(px[0]);
    px[0] = load_x(min(t0 + 1, last), 0);
    form_y(py[0], mul, A[0]);
    load_y(min(t0 + 2, last), py[0]);
    for (int t = t0; t <= last; t += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
          const int k = (n + 1) % NJ;
          const Frag next = form_x(px[k]);
          px[k] = load_x(min(t + u + (k == 0 ? 2 : 1), last), k);
          products(A[u], B, n);
          B = next;
        }
        const int v = 1 - u;
        form_y(py[v], t + u + 1 <= last ? mul : 0.0f, A[v]);
        load_y(min(t + u + 3, last), py[v]);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    static_assert(kS == 2 && kAhead == 2, "two steps a stage");
    const int stages = steps / kS;
    store_stage(0);
    load_stage(1);
    form_y(py[0], mul, A[0]);
    load_y(min(t0 + 2, last), py[0]);
    __syncthreads();
    for (int s = 0; s < stages; ++s) {
      const uint4* src = buf + (s & 1) * kBuf + lane;
      auto read_x = [&](int b) -> Frag {
        const uint4* q = src + b * kPlanes * kWave;
        Frag f;
        f.hi = q[0];
        f.lo = kPlanes > 1 ? q[kWave] : f.hi;
        return f;
      };
      Frag B = read_x(0);
#pragma unroll
      for (int u = 0; u < kS; ++u) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
          const int b = u * NJ + n + 1;
          const Frag next = b < kS * NJ ? read_x(b) : B;
          products(A[u], B, n);
          B = next;
        }
        // the next step's rows, and this wave's share of the next stage's columns
        const int v = 1 - u;
        form_y(py[v], mul, A[v]);
        load_y(min(t0 + s * kS + u + 3, last), py[v]);
#pragma unroll
        for (int k = u * kShare / kS; k < (u + 1) * kShare / kS; ++k) {
          store_block(s + 1, k);
          load_block(s + 2, k);
        }
        interleave();
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    }
  }

  // An infinite amplitude has no scale: such a call takes the sum term by term,
  // cos(X + Y) A, so that its infinities and NaNs are the direct sum's.  A NaN makes
  // every pixel NaN and needs no sum.
  if (MODE == kHalfF16x3 && !finite_bits(m)) {
    for (int e = grp * kWave + lane; e < MI * 32 * NJ * 32; e += KS * kWave) {
      const int row = y0 + e / (NJ * 32), col = x0 + e % (NJ * 32);
      if (row >= ny || col >= nx) continue;
      float v = nan_bits(m) ? __builtin_nanf("") : 0.0f;
      for (int64_t q = first / 4; !nan_bits(m) && q < min(first + per_slice, npad) / 4; ++q) {
        const float4 Y = static_cast<const float4*>(o.yq)[q * o.rows_y + row];
        const float4 X = XTAB ? static_cast<const float4*>(o.xq)[q * o.cols_x + col]
                              : quad_phases(o.rec, q, (float)col);
        const float4 a = *reinterpret_cast<const float4*>(o.amp + q * 4);
        v = __builtin_fmaf(a.x, cos_rev(X.x + Y.x), v);
        v = __builtin_fmaf(a.y, cos_rev(X.y + Y.y), v);
        v = __builtin_fmaf(a.z, cos_rev(X.z + Y.z), v);
        v = __builtin_fmaf(a.w, cos_rev(X.w + Y.w), v);
      }
      const int64_t idx = (int64_t)row * nx + col;
      out[idx] = v;
      if constexpr (RES) res[idx] = v - tgt[idx];
    }
    return;
  }

  // The groups' sums, kChunk registers of every wave a round through LDS: each
  // wave of a group then adds the KS copies of its kOwn registers in group order
  // and stores those pixels, so the sums, the target's loads and the stores are
  // spread over all waves.  (One wave storing alone took 30 us longer with a
  // target at 1920x1024.)
  float* sums = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int h = 0; h < kRounds; ++h) {
    const int mine = h * kChunk + grp * kOwn;  // first owned register, of block mine / 16
    if (WM > 1 || h > 0) __syncthreads();
#pragma unroll
    for (int c = 0; c < kChunk; c += kVec) {
      float* d = sums + (((grp * WM + w) * kChunk + c) * kWave + lane * kVec);
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        const int q = h * kChunk + c + e;
        d[e] = acc[q / 16 / NJ][q / 16 % NJ][q % 16];
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kOwn; c += kVec) {
      const int q = mine + c, r = q % 16;
      const int row = y0 + q / 16 / NJ * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
      const int col = x0 + q / 16 % NJ * 32 + l32;
      const int64_t idx = (int64_t)row * nx + col;
      float t[kVec], v[kVec];
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        t[e] = RES && row + e < ny && col < nx ? tgt[idx + (int64_t)e * nx] : 0.0f;
        v[e] = 0.0f;
      }
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const float* d = sums + (((k * WM + w) * kChunk + grp * kOwn + c) * kWave + lane * kVec);
#pragma unroll
        for (int e = 0; e < kVec; ++e) v[e] = k == 0 ? d[e] : v[e] + d[e];
      }
#pragma unroll
      for (int e = 0; e < kVec; ++e)
        if (row + e < ny && col < nx) {
          v[e] *= undo;
          out[idx + (int64_t)e * nx] = v[e];
          if constexpr (RES) res[idx + (int64_t)e * nx] = v[e] - t[e];
        }
    }
  }
}

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Largest |A|, as float bits, of each of kWave parts of the points.
__global__ __launch_bounds__(256) void contract_amax_kernel(const float* __restrict__ a, int64_t n,
                                                            unsigned* __restrict__ amax) {
  __shared__ unsigned red[4];
  unsigned m = 0;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n; k += 256 * kWave)
    m = max(m, __float_as_uint(fabsf(a[k])));
  m = group_max<256>(m, red);
  if (threadIdx.x == 0) amax[blockIdx.x] = m;
}

// Both tables, the amplitudes and (without an x table) the x records in one
// launch.  A workgroup is 16 points (blockIdx.x) and kTabRows coordinates
// (blockIdx.y: y slices, then x slices).  Lane l of wave w takes point
// 4 w + l % 4 of the 16 and coordinates l / 4, l / 4 + 16, ..., so a store is
// 256 consecutive bytes.
template <int MODE>
__global__ __launch_bounds__(256) void contract_fwd_tables_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int64_t n, double pitch, double wavelength, int yslices,
    int rows_y, int cols_x, uint32_t* __restrict__ yq, uint32_t* __restrict__ xq,
    float* __restrict__ rec, float* __restrict__ amp, unsigned* __restrict__ amax) {
  __shared__ unsigned red[4];
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int e = lane & 3;
  const int64_t j = q * 4 + e;
  const bool is_y = (int)blockIdx.y < yslices;
  const int slice = is_y ? (int)blockIdx.y : (int)blockIdx.y - yslices;
  float mul = 1.0f;
  if ((MODE == kHalfF16 || MODE == kHalfBF16) && is_y) {
    // Few points: every y workgroup takes the largest |A| itself, n words from
    // the cache; else the maxima of contract_amax_kernel are there.
    unsigned m = 0;
    if (n <= kAmaxInline) {
      const int64_t n4 = n / 4;
      for (int64_t k = threadIdx.x; k < n4; k += 256) {
        const f32x4u v = reinterpret_cast<const f32x4u*>(a)[k];
        m = max(m, max(max(__float_as_uint(fabsf(v.x)), __float_as_uint(fabsf(v.y))),
                       max(__float_as_uint(fabsf(v.z)), __float_as_uint(fabsf(v.w)))));
      }
      if (threadIdx.x < n - 4 * n4) m = max(m, __float_as_uint(fabsf(a[4 * n4 + threadIdx.x])));
      m = group_max<256>(m, red);
      if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kWave) amax[threadIdx.x] = m;
    } else {
      m = group_max<kWave>(amax[lane], red);
    }
    float undo;
    operand_scale<MODE>(m, mul, undo);
  }
  // The records, one a thread of the first sixteen.  (Formed by every thread, the
  // launch took 20.7 us where it takes 19.9 at 1920x1080, N = 8192 in f16x3; in f16,
  // with max |A| a word a load, 33.7 and 26.3.)
  __shared__ PointRecord records[16];
  if (threadIdx.x < 16)
    records[threadIdx.x] = point_record(x, y, z, a, (int64_t)blockIdx.x * 16 + threadIdx.x, n,
                                        pitch, wavelength);
  __syncthreads();
  const PointRecord r = records[(threadIdx.x >> 6) * 4 + e];
  if (blockIdx.y == 0 && lane < 4) {
    amp[j] = r.a;
    if (rec) {
      float* d = rec + q * 20 + e;
      d[0] = r.xc;
      d[4] = r.ph;
      d[8] = r.pl;
      d[12] = r.xb;
      d[16] = r.xd;
    }
  }
  const float A = r.a * mul;
  const int rows = is_y ? rows_y : cols_x;
  const float c = is_y ? r.yc : r.xc, b = is_y ? r.yb : r.xb, d = is_y ? r.yd : r.xd;
  uint32_t* dst = (is_y ? yq : xq) + (q * rows) * 4 + e;
#pragma unroll 4
  for (int i = 0; i < kTabRows / 16; ++i) {
    const int h = slice * kTabRows + (lane >> 2) + 16 * i;
    if (h >= rows) break;
    const float ph = axis_phase((float)h, c, r.ph, r.pl, b, d);
    if constexpr (MODE == kHalfF16x3) {
      dst[h * 4] = __float_as_uint(ph);
    } else if constexpr (MODE == kF32) {
      const float cs = cos_rev(ph), sn = sin_rev(ph);
      float* d2 = reinterpret_cast<float*>(is_y ? yq : xq) +
                  (e >> 1) * ((int64_t)gridDim.x * 16 * rows) + (q * rows + h) * 4 + (e & 1) * 2;
      *reinterpret_cast<float2*>(d2) = is_y ? make_float2(A * cs, -(A * sn)) : make_float2(cs, sn);
    } else {
      const float cs = cos_rev(ph), sn = sin_rev(ph);
      dst[h * 4] = is_y ? pack16<MODE>(A * cs, -(A * sn)) : pack16<MODE>(cs, sn);
    }
  }
}

// Few points on a small hologram, in one launch without tables: a call of two
// launches there is bound by them (256x256, N = 64: 14.3 us a call, 11.3 here).
// A workgroup is 32 x 32 pixels and eight waves.  It forms the records of up to
// 512 points at a time in LDS, one a thread; wave w takes steps w, w + 8, ... of
// eight points, each lane the phases of its four points at its row and its
// column, from records that all lanes of a half read together (broadcasts).  Tiles of one block form every
// phase once per 32 pixels, 0.9 instructions an interaction, which is why many
// points or large holograms take tables and larger tiles.
constexpr int kDirectPoints = 512;
template <int MODE, bool RES>
__global__ __launch_bounds__(512) void contract_fwd_direct_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int n, double pitch, double wavelength, int nx, int ny,
    unsigned tiles_x, float* __restrict__ out, const float* __restrict__ tgt,
    float* __restrict__ res) {
  constexpr int kWaves = 8;
  __shared__ float4 lds[kWaves * 16 * kWave / 4];  // the records, later the waves' sums
  __shared__ unsigned red[kWaves];
  static_assert(9 * kDirectPoints * sizeof(float) <= sizeof(lds), "the records fit");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int half = lane >> 5, l32 = lane & 31;
  const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);
  const int y0 = (int)(tile / tiles_x) * 32, x0 = (int)(tile % tiles_x) * 32;
  const float row = (float)(y0 + l32), col = (float)(x0 + l32);

  PointRecord r = point_record(x, y, z, a, threadIdx.x, n, pitch, wavelength);
  unsigned m = 0;
  float mul = 1.0f, undo = 1.0f;
  if (MODE != kF32) {
    m = __float_as_uint(fabsf(r.a));
    for (int j = kDirectPoints + threadIdx.x; j < n; j += kDirectPoints)
      m = max(m, __float_as_uint(fabsf(a[j])));
    m = group_max<512>(m, red);
    operand_scale<MODE>(m, mul, undo);
  }
  floatx16 acc;
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.0f;
  float direct[2] = {0.0f, 0.0f};  // this thread's two pixels, of a sum without a scale
  const int sum_at = (threadIdx.x >> 6) * 2;  // their registers: sum_at and sum_at + 1

  float* recs = reinterpret_cast<float*>(lds);
  if (nan_bits(m)) direct[0] = direct[1] = __builtin_nanf("");
  for (int base = 0; base < n; base += kDirectPoints) {
    if (base > 0) {
      r = point_record(x, y, z, a, base + threadIdx.x, n, pitch, wavelength);
      __syncthreads();
    }
    float* d = recs + threadIdx.x;
    d[0 * kDirectPoints] = r.ph;
    d[1 * kDirectPoints] = r.pl;
    d[2 * kDirectPoints] = r.yc;
    d[3 * kDirectPoints] = r.yb;
    d[4 * kDirectPoints] = r.yd;
    d[5 * kDirectPoints] = r.xc;
    d[6 * kDirectPoints] = r.xb;
    d[7 * kDirectPoints] = r.xd;
    d[8 * kDirectPoints] = r.a;
    __syncthreads();
    const int here = min(kDirectPoints, n - base);
    if (MODE == kHalfF16x3 && !finite_bits(m)) {
      for (int j = 0; j < here && !nan_bits(m); ++j) {
        const float* q = recs + j;
        const float X = axis_phase(col, q[5 * kDirectPoints], q[0], q[kDirectPoints],
                                   q[6 * kDirectPoints], q[7 * kDirectPoints]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int k = sum_at + e;
          const float h = (float)(y0 + (k >> 2) * 8 + half * 4 + (k & 3));
          const float Y = axis_phase(h, q[2 * kDirectPoints], q[0], q[kDirectPoints],
                                     q[3 * kDirectPoints], q[4 * kDirectPoints]);
          direct[e] = __builtin_fmaf(q[8 * kDirectPoints], cos_rev(X + Y), direct[e]);
        }
      }
      continue;
    }
    for (int t = wave; t * 8 < here; t += kWaves) {
      const float4* q = lds + 2 * t + half;
      constexpr int kQuads = kDirectPoints / 4;
      const float4 ph = q[0], pl = q[kQuads];
      auto phases = [&](float h, const float4& c, const float4& b, const float4& d) {
        return make_float4(axis_phase(h, c.x, ph.x, pl.x, b.x, d.x),
                           axis_phase(h, c.y, ph.y, pl.y, b.y, d.y),
                           axis_phase(h, c.z, ph.z, pl.z, b.z, d.z),
                           axis_phase(h, c.w, ph.w, pl.w, b.w, d.w));
      };
      const float4 Y = phases(row, q[2 * kQuads], q[3 * kQuads], q[4 * kQuads]);
      const float4 X = phases(col, q[5 * kQuads], q[6 * kQuads], q[7 * kQuads]);
      const float4 A = q[8 * kQuads];
      const Frag P = frag_of_phases<MODE>(Y, make_float4(A.x * mul, A.y * mul, A.z * mul, A.w * mul));
      const Frag Q = frag_of_phases<MODE>(X);
      auto part = [&](auto k) { acc = mfma_part<MODE, decltype(k)::value>(P, Q, acc); };
      parts(part, std::make_integer_sequence<int, mfmas_per_step(MODE)>{});
    }
  }

  // The waves' sums in wave order; thread t stores two pixels.
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) recs[(wave * 16 + k) * kWave + lane] = acc[k];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int k = sum_at + e;
    float v = recs[k * kWave + lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += recs[(w * 16 + k) * kWave + lane];
    v *= undo;
    if (MODE == kHalfF16x3 && !finite_bits(m)) v = direct[e];
    const int yy = y0 + (k >> 2) * 8 + half * 4 + (k & 3), xx = x0 + l32;
    if (yy < ny && xx < nx) {
      const int64_t at = (int64_t)yy * nx + xx;
      out[at] = v;
      if constexpr (RES) res[at] = v - tgt[at];
    }
  }
}

template <int MODE, int MI, int NJ, int WM, int KS>
hipError_t launch_shape(const Plan& p, const ContractFwd& c, float* out, const float* tgt,
                        float* res, hipStream_t s) {
  const int64_t tiles_x = (p.nx + NJ * 32 - 1) / (NJ * 32);
  const int64_t tiles_y = (p.ny + WM * MI * 32 - 1) / (WM * MI * 32);
  const int64_t tiles = tiles_x * tiles_y;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  if (tiles * c.slices > 0x7fffffff) return hipErrorInvalidValue;
  const FwdOperands o{c.yq, c.xtab ? c.xq : nullptr, c.rec, c.amp, c.rows_y, c.cols_x};
  constexpr int kUnit = KS == 1 ? 16 : 64;  // points
  const int per_slice = (int)((p.npad / kUnit + c.slices - 1) / c.slices * kUnit);
  const bool one = c.slices == 1;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles * c.slices)), dim3(kWave * WM * KS), 0, s, o,
                       (int)p.npad, p.nx, p.ny, (unsigned)tiles_x, (unsigned)tiles, per_slice,
                       c.amax, one ? out : c.planes, tgt, res);
  };
  if (c.xtab) {
    if (res && one)
      go(contract_fwd_kernel<MODE, MI, NJ, WM, KS, true, true>);
    else
      go(contract_fwd_kernel<MODE, MI, NJ, WM, KS, true, false>);
  } else if constexpr (MODE == kHalfF16x3 && KS > 1) {
    if (res && one)
      go(contract_fwd_kernel<MODE, MI, NJ, WM, KS, false, true>);
    else
      go(contract_fwd_kernel<MODE, MI, NJ, WM, KS, false, false>);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// I = the sum of the slices' planes in order, and I - T with a target.
__global__ __launch_bounds__(256) void contract_fwd_sum_kernel(const float* __restrict__ planes,
                                                               int slices, int64_t count,
                                                               float* __restrict__ out,
                                                               const float* __restrict__ tgt,
                                                               float* __restrict__ res) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  float v = planes[i];
#pragma unroll 8
  for (int k = 1; k < slices; ++k) v += planes[k * count + i];
  out[i] = v;
  if (res) res[i] = v - tgt[i];
}

// I += plane, and I - T with a target.
__global__ __launch_bounds__(256) void contract_fwd_add_kernel(const float* __restrict__ plane,
                                                               int64_t count,
                                                               float* __restrict__ out,
                                                               const float* __restrict__ tgt,
                                                               float* __restrict__ res) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float v = out[i] + plane[i];
  out[i] = v;
  if (res) res[i] = v - tgt[i];
}

// Tile shapes <MI, NJ, WM, KS>: pixels per workgroup and the terms of its time
// on this GPU: microseconds per launch beside the loop; per round of 256 workgroups
// (one a CU) for its sums and stores, which count where few points light many pixels
// (below; us with the first shape and with the one that the other terms prefer:
// 6029x4883, N = 9 in bf16: 45 and 91; 3840x2160, N = 256: 28 and 37; N = 64 in FP32: 39
// and 63); and per 1000 points and round, for f16x3, for the single planes and for FP32, each in a
// launch of one round and of more.  Larger tiles form fewer operands per
// product (per pixel <2, 4, 2, 2> takes 0.7 of <2, 2, 1, 4>'s time and 0.4 of
// <1, 1, 1, 8>'s); smaller ones and more point groups put a small hologram on
// more CUs.  Measured at 50 random sizes (64 to 3840 by 64 to 2160, 64 to 65,536
// points), the choice is within 4% of the best shape on average, 21% at most.
struct Shape {
  int rows, cols, groups;
  float fixed, round, split_one, split, single_one, single, f32_one, f32;
};
constexpr Shape kShapes[] = {
    {128, 128, 2, 9.5f, 2.2f, 47.0f, 47.0f, 29.0f, 29.0f, 132.0f, 140.0f},  // <2, 4, 2, 2>
    {64, 128, 8, 9.0f, 5.5f, 26.0f, 26.0f, 12.0f, 12.0f, 77.0f, 77.0f},   // <2, 4, 1, 8>
    {64, 64, 4, 7.0f, 1.1f, 18.5f, 15.5f, 10.0f, 7.8f, 40.6f, 38.5f},     // <2, 2, 1, 4>
    {64, 64, 8, 8.0f, 2.5f, 15.2f, 16.0f, 8.0f, 8.0f, 36.6f, 39.5f},      // <2, 2, 1, 8>
    {32, 64, 8, 6.5f, 1.3f, 10.5f, 10.3f, 6.2f, 5.6f, 19.6f, 20.5f},      // <1, 2, 1, 8>
    {32, 32, 8, 5.0f, 0.8f, 7.5f, 7.0f, 4.2f, 4.0f, 11.0f, 10.6f},        // <1, 1, 1, 8>
};

// Shape and slices for plan p, and the least time in microseconds without the stores
// (which use_direct and plan_chunks compare with times without them).  Cutting the
// points into slices (as far as the plan has room for their planes) puts a small
// hologram of many points on more CUs, at one more launch (6 us) and the planes' traffic (at 3 TB/s); a slice
// has at least 512 points.  (128x96, N = 60000: 410 us in one slice, 36 in 21.)
// The sums are cut into at least min_parts parts (slices times point groups),
// which bounds the error of the FP32 additions: it grows as the square root of
// a part's length (3332x341, N = 60771: 2.97e-6 of the result in 2 parts,
// 4.3e-7 in 64).  min_parts is the plan's K splits for f16x3 and FP32 and 1 for the
// compensated variant, whose direct form is one chain of all points (1.5e-8 sqrt(N)
// of the result, 3.7e-6 there).
int choose_shape(int64_t npad, int32_t nx, int32_t ny, int mode, int64_t max_slices,
                 int64_t min_parts, int& slices, float& best_time) {
  int best = 0;
  float best_cost = 0.0f;
  best_time = 0.0f;
  slices = 1;
  const int64_t units = npad / 64;  // points are cut in units of 64
  const int64_t most = mode == kF32 ? 4096 : 1024;  // workgroups of a sliced launch
  const bool count_stores =
      mode == kF32         ? npad <= 64
      : mode == kHalfF16x3 ? npad <= 512 && (int64_t)nx * ny > int64_t(1) << 23
                           : npad <= 2048 && (int64_t)nx * ny > int64_t(5) << 20;
  const float plane_us = (float)nx * (float)ny * (8.0f / 3e6f);
  for (int k = 0; k < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++k) {
    const Shape& q = kShapes[k];
    const int64_t tiles = (((int64_t)nx + q.cols - 1) / q.cols) * (((int64_t)ny + q.rows - 1) / q.rows);
    for (int64_t want = 1; want <= max_slices || want == 1; want += want < 4 ? 1 : want / 2) {
      const int64_t per = (units + want - 1) / want, n = (units + per - 1) / per;  // none empty
      const bool few = n * q.groups < min_parts && n < max_slices && n < units;
      if (want > 1 && !few && (units < 8 * want || tiles * want > most) && best_time > 0.0f) break;
      if (few) continue;
      // (HIP takes 2^32 - 1 threads a launch; the first shape's stay below on any
      // hologram that fits the memory)
      if (k > 0 && tiles * n * q.groups * kWave > 0xffffffffll) break;
      const int64_t rounds = (tiles * n + 255) / 256;
      const float per_k = mode == kHalfF16x3 ? (rounds == 1 ? q.split_one : q.split)
                          : mode == kF32     ? (rounds == 1 ? q.f32_one : q.f32)
                                             : (rounds == 1 ? q.single_one : q.single);
      const float stores = count_stores ? (float)rounds * q.round : 0.0f;
      const float time = q.fixed + (float)rounds * (float)(per * 64) * 1e-3f * per_k +
                         (n > 1 ? 6.0f + (float)n * plane_us : 0.0f);
      if (best_time == 0.0f || time + stores < best_cost) {
        best = k;
        best_cost = time + stores;
        slices = (int)n;
      }
      best_time = best_time == 0.0f ? time : std::min(best_time, time);
    }
  }
  return best;
}

template <int MODE>
hipError_t launch_mode(const Plan& p, const ContractFwd& c, float* out, const float* tgt,
                       float* res, hipStream_t s) {
  switch (c.shape) {
    case 0: return launch_shape<MODE, 2, 4, 2, 2>(p, c, out, tgt, res, s);
    case 1: return launch_shape<MODE, 2, 4, 1, 8>(p, c, out, tgt, res, s);
    case 2: return launch_shape<MODE, 2, 2, 1, 4>(p, c, out, tgt, res, s);
    case 3: return launch_shape<MODE, 2, 2, 1, 8>(p, c, out, tgt, res, s);
    case 4: return launch_shape<MODE, 1, 2, 1, 8>(p, c, out, tgt, res, s);
    case 5: return launch_shape<MODE, 1, 1, 1, 8>(p, c, out, tgt, res, s);
    // (us at 1 x 1, 1 x 2 and 2 x 2 blocks: 448x336, N = 42208: FP32 332, 362, 431; f16x3
    // 240, 216, 222; f16 119, 104, 93.  146x121, N = 25918: FP32 62, 67, 74.)
    case kOrdered: {
      constexpr int kSide = MODE == kF32 ? 1 : 2;
      return launch_shape<MODE, kSide, kSide, 1, 1>(p, c, out, tgt, res, s);
    }
    default: return hipErrorInvalidValue;
  }
}

// Whether one launch of contract_fwd_direct_kernel is faster than the tables'
// launch and the shape that takes `tiled` us.  It takes 4.5 us and, for each
// round of 256 tiles, 0.45 and the given time per 1000 points; the tables take
// 3.5 us and more.  (us a call, tables and direct: 256x256, N = 64: 14.3 and 11.3;
// N = 1024: 15.2 and 14.9; N = 2048: 17.3 and 26.5; 1920x1080, N = 64: 20.0 and
// 12.7; N = 128: 14.3 and 17.5.)  Beyond two rounds of records it loses to the
// tables, and its eight partial sums a pixel become longer than theirs.
bool use_direct(int64_t n, int32_t nx, int32_t ny, int mode, float tiled) {
  if (n > 2 * kDirectPoints) return false;
  const int64_t tiles = ((int64_t)nx + 31) / 32 * (((int64_t)ny + 31) / 32);
  if (tiles > 1 << 20) return false;  // (a grid of 2^32 threads at most)
  const float rounds = (float)((tiles + 255) / 256);
  const float per_k = mode == kHalfF16x3 ? 9.2f : mode == kF32 ? 13.2f : 7.0f;
  return 4.5f + rounds * (0.45f + (float)n * 1e-3f * per_k) < tiled + 3.5f;
}

// Without room for the column table of all points, the row table's region holds
// both tables of a part of them and a plane for that part's sum, and the points can
// be taken in chunks.  A pass takes its shape's time, 12 us for its launches and
// the planes' traffic; forming the x-phases in the kernel takes about 1.3 times
// `inline_us`, the shape's time with tables.  (us a call, formed in the kernel and
// in chunks: 1920x1080, N = 65536: 2357 and 1871; 3840x800, N = 40000: 3002 and
// 1934; 2011x81, N = 96630: 517 and, in 23 chunks, 1184.)  A rule on the plan alone,
// so every entry point takes the same way.
constexpr int64_t kMinChunk = 4096;
void plan_chunks(const Plan& p, const Workspace& w, float inline_us, ContractFwd& c) {
  const int64_t room = (int64_t)c.rows_y * p.npad;  // words
  const int64_t pixels = (int64_t)p.nx * p.ny, units = p.npad / 64;
  if (pixels > 0x7fffffff) return;  // (the planes' kernels take a thread a pixel)
  for (int64_t k = 1 + (c.cols_x + c.rows_y - 1) / c.rows_y;; ++k) {
    const int64_t chunk = (units + k - 1) / k * 64;
    if (chunk < kMinChunk) return;
    const int64_t left = room - chunk * ((int64_t)c.rows_y + c.cols_x) - pixels;
    if (left < 0) continue;
    int slices;
    float time;
    const int shape = choose_shape(chunk, p.nx, p.ny, c.mode, left / pixels, 1, slices, time);
    const float passes = (float)((p.npad + chunk - 1) / chunk);
    if (passes * (time + 12.0f + (float)pixels * (12.0f / 4e6f)) > 1.3f * inline_us) return;
    c.shape = shape;
    c.slices = slices;
    c.chunk = chunk;
    c.xtab = true;
    c.xq = w.ytab + chunk * c.rows_y;
    c.planes = w.ytab + chunk * ((int64_t)c.rows_y + c.cols_x);  // a pass's sum, its slices
    return;
  }
}

}  // namespace

int contract_fwd_slices(int64_t npad, int32_t nx, int32_t ny) {
  int slices;
  float time;
  (void)choose_shape(npad, nx, ny, kHalfF16x3, INT64_MAX / 2, 1, slices, time);
  return slices;
}

bool plan_contract_fwd(const Plan& p, const Workspace& w, ContractFwd& c) {
  c = ContractFwd{};
  if (p.op != 0) return false;
  if (p.variant == 1) {
    // Up to 8 points (one step of the contraction) stay with the direct kernel:
    // both take the time of their launches there (17 us a call at 101x121,
    // N = 1), and of a single point the direct form keeps the exact eightfold
    // symmetry, since A multiplies the whole cosine and not the row factor.
    // Sums that keep the order of the points are its own too: the matrix cores add
    // 16 products at a time.
    if (p.n <= 8 || ordered_sum(p.n, p.nx, p.ny)) return false;
    c.mode = kHalfF16x3;
    c.rows_y = p.groups * kCompRows;
    c.cols_x = p.fwd_gx * kWave;
    c.xtab = w.xtab != nullptr;
    c.yq = w.ytab;
    c.xq = w.xtab;
  } else {
    c.mode = p.variant == 2 ? kF32 : p.variant == 3 ? kHalfF16x3 : p.variant == 4 ? kHalfF16 : kHalfBF16;
    c.rows_y = p.nyp;
    c.cols_x = p.nxp;
    c.xtab = true;
    c.yq = p.variant == 2 ? w.sep_y : w.htab_y;
    c.xq = p.variant == 2 ? w.sep_x : w.htab_x;
  }
  c.rec = (float4*)w.xrec;
  c.amp = w.amp;
  c.amax = w.hmax;
  if (p.variant != 1 && ordered_splits(p.n, p.nx, p.ny)) {
    c.shape = kOrdered;
    c.slices = p.sep_splits;
    c.planes = w.sep_c;
    return true;
  }
  // Planes of the point slices: the plan's own, the split planes of the
  // separable plans, or the y records (which this path does not use).
  const int64_t pixels = (int64_t)p.nx * p.ny;
  const int64_t in_rec = p.npad * kAxisRec / pixels;
  const int64_t in_sep = w.sep_c ? p.sep_splits * ((int64_t)p.nxp * p.nyp) / pixels : 0;
  int64_t room = in_rec;
  c.planes = w.yrec;
  if (p.fwd_planes > 0) {
    room = p.fwd_planes;
    c.planes = w.planes;
  } else if (in_sep > in_rec) {
    room = in_sep;
    c.planes = w.sep_c;
  }
  // The f16x3 and f32 separable variants sum in at least as many parts as their
  // plan's K splits.
  const int64_t parts = p.variant == 3 || p.variant == 2 ? p.sep_splits : 1;
  float time;
  c.shape = choose_shape(p.npad, p.nx, p.ny, c.mode, room, parts, c.slices, time);
  c.direct = use_direct(p.n, p.nx, p.ny, c.mode, time);
  if (p.variant == 1 && p.comp_wide && !c.direct) plan_chunks(p, w, time, c);
  // The single planes are bound by their operand loads: tables that exceed the 256
  // MB Infinity Cache are formed and read in passes that fit it, where there is
  // room for a pass's plane.  (us a call in f16, in one pass, of 96 MB and of 192 MB:
  // 1673x658, N = 51542: 601, 525, 443; 1920x1080, N = 65536: 915, 848, 806;
  // 1382x471, N = 36660: 271, 259, 239.  f16x3 and FP32, with more work an operand,
  // gain nothing or lose.)
  constexpr int64_t kCached = int64_t(256) << 20, kPassBytes = int64_t(192) << 20;
  const int64_t point_bytes = ((int64_t)c.rows_y + c.cols_x) * 4;  // tables, a point
  if ((c.mode == kHalfF16 || c.mode == kHalfBF16) && point_bytes * p.npad > kCached && room >= 2 &&
      pixels <= 0x7fffffff) {
    const int64_t passes = (point_bytes * p.npad + kPassBytes - 1) / kPassBytes;
    const int64_t chunk = (p.npad / 64 + passes - 1) / passes * 64;
    if (chunk >= kMinChunk) {
      c.chunk = chunk;
      c.shape = choose_shape(chunk, p.nx, p.ny, c.mode, room - 1, 1, c.slices, time);
    }
  }
  return true;
}

hipError_t launch_contract_fwd_tables(const Plan& p, const ContractFwd& c, const float* x,
                                      const float* y, const float* z, const float* a,
                                      double pitch, double wavelength, hipStream_t s) {
  const int yslices = (c.rows_y + kTabRows - 1) / kTabRows;
  const int xslices = c.xtab ? (c.cols_x + kTabRows - 1) / kTabRows : 0;
  const dim3 grid((unsigned)(p.npad / 16), (unsigned)(yslices + xslices));
  const bool single = c.mode == kHalfF16 || c.mode == kHalfBF16;
  if ((single && p.n > kAmaxInline) || (c.mode == kHalfF16x3 && c.shape == kOrdered))
    hipLaunchKernelGGL(contract_amax_kernel, dim3(kWave), dim3(256), 0, s, a, p.n, c.amax);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, x, y, z, a, p.n, pitch, wavelength, yslices,
                       c.rows_y, c.cols_x, (uint32_t*)c.yq, (uint32_t*)c.xq,
                       c.xtab ? (float*)nullptr : (float*)c.rec, c.amp, c.amax);
  };
  if (c.mode == kHalfF16x3)
    go(contract_fwd_tables_kernel<kHalfF16x3>);
  else if (c.mode == kF32)
    go(contract_fwd_tables_kernel<kF32>);
  else if (c.mode == kHalfF16)
    go(contract_fwd_tables_kernel<kHalfF16>);
  else
    go(contract_fwd_tables_kernel<kHalfBF16>);
  return hipGetLastError();
}

hipError_t launch_contract_direct(const Plan& p, const ContractFwd& c, const float* x,
                                  const float* y, const float* z, const float* a, double pitch,
                                  double wavelength, float* out, const float* target,
                                  float* residual, hipStream_t s) {
  const int64_t tiles_x = (p.nx + 31) / 32, tiles = tiles_x * ((p.ny + 31) / 32);
  if (tiles > 0x7fffffff || p.n > 0x7fffffff - kDirectPoints) return hipErrorInvalidValue;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(512), 0, s, x, y, z, a, (int)p.n, pitch,
                       wavelength, p.nx, p.ny, (unsigned)tiles_x, out, target, residual);
  };
  auto either = [&](auto mode) {
    constexpr int kMode = decltype(mode)::value;
    if (residual)
      go(contract_fwd_direct_kernel<kMode, true>);
    else
      go(contract_fwd_direct_kernel<kMode, false>);
  };
  if (c.mode == kHalfF16x3)
    either(std::integral_constant<int, kHalfF16x3>{});
  else if (c.mode == kF32)
    either(std::integral_constant<int, kF32>{});
  else if (c.mode == kHalfF16)
    either(std::integral_constant<int, kHalfF16>{});
  else
    either(std::integral_constant<int, kHalfBF16>{});
  return hipGetLastError();
}

hipError_t launch_contract_fwd(const Plan& p, const ContractFwd& c, float* out,
                               const float* target, float* residual, hipStream_t s) {
  hipError_t e;
  if (c.mode == kHalfF16x3)
    e = launch_mode<kHalfF16x3>(p, c, out, target, residual, s);
  else if (c.mode == kF32)
    e = launch_mode<kF32>(p, c, out, target, residual, s);
  else if (c.mode == kHalfF16)
    e = launch_mode<kHalfF16>(p, c, out, target, residual, s);
  else
    e = launch_mode<kHalfBF16>(p, c, out, target, residual, s);
  if (e != hipSuccess || c.slices == 1) return e;
  const int64_t count = (int64_t)p.nx * p.ny;
  hipLaunchKernelGGL(contract_fwd_sum_kernel, dim3(grid_blocks(count, 256)), dim3(256), 0, s,
                     c.planes, c.slices, count, out, target, residual);
  return hipGetLastError();
}

hipError_t launch_contract_chunks(const Plan& p, const ContractFwd& c, const float* x,
                                  const float* y, const float* z, const float* a, double pitch,
                                  double wavelength, float* out, const float* target,
                                  float* residual, hipStream_t s) {
  const int64_t pixels = (int64_t)p.nx * p.ny;
  ContractFwd part = c;
  part.planes = c.planes + pixels;
  for (int64_t first = 0; first < p.npad; first += c.chunk) {
    Plan q = p;
    q.npad = std::min(c.chunk, p.npad - first);
    q.n = std::min(q.npad, p.n - first);
    const int64_t units = q.npad / 64, per = (units + c.slices - 1) / c.slices;
    part.slices = (int)((units + per - 1) / per);  // none empty in a shorter last pass
    hipError_t e = launch_contract_fwd_tables(q, part, x + first, y + first, z + first, a + first,
                                              pitch, wavelength, s);
    if (e == hipSuccess)
      e = launch_contract_fwd(q, part, first == 0 ? out : c.planes, nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    if (first > 0)
      hipLaunchKernelGGL(contract_fwd_add_kernel, dim3(grid_blocks(pixels, 256)), dim3(256), 0, s,
                         c.planes, pixels, out, first + c.chunk < p.npad ? nullptr : target,
                         first + c.chunk < p.npad ? nullptr : residual);
  }
  return hipGetLastError();
}

}  // namespace cgh
