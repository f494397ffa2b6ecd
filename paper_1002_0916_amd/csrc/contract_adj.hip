// Adjoint of Eq. (1) (Section 1) as two contractions on the matrix cores
// (contract.h), with their operands formed in the kernel and their results
// folded there:
//
//   U_j(x) = sum_y G cY, V_j(x) = sum_y G sY        (x part: u = x, v = y)
//   U_j(y) = sum_x G cX, V_j(y) = sum_x G sX        (y part: u = y, v = x)
//
// and with w_j(u) = s U + c V, (c, s) the cosine and sine of the phase of point
// j at u, the sums of the adjoint (adjoint.hip) are
//
//   Sc = sum_x (c U - s V)                    Sx = sum_x dx w, Sy = sum_y dy w
//   Sr = sum_x dx^2 w + sum_y dy^2 w.
//
// A workgroup takes 128 points and, one after the other, the tiles of 128
// coordinates u of its column group, over its slice of v.  Each of its four
// waves has 32 points (one per lane, in both halves of the wave), so both
// results of a point are in one lane, U in one set of accumulators and V in
// another: the fold over u runs inside the lane, and only the two halves of the
// wave are added across lanes.  (Accumulator register r of lane l is u = (r /
// 4) * 8 + (l / 32) * 4 + r % 4 of its block of 32, so a lane's four registers
// are one quad of the u table.)
//
// Operands: a wave forms its points' cosines and sines at 16 v per step from
// the phase table (or from its point's record) in registers, in the matrix
// cores' layout (lane l: v = (l / 32) * 8 .. + 7).  G is read as FP32, scaled,
// split and left in LDS by all four waves, 32 v by 128 u per stage, double
// buffered; slot s of a 1 KB block holds lane s ^ (4 * octet) of each half, so
// that neither the reads nor the writes of either part meet a bank twice.
//
// FP32 (8 flops per interaction on the FP32 matrix cores, which bound it) reads
// the same tables of phases; its G goes through LDS as it is.  1024x1024, N =
// 4096: 310 us a call where two tiled products of operand tables with a fold took
// 358.
#include "contract.h"
#include "records.h"

namespace cgh {

namespace {

constexpr int kAdjTile = 128;   // coordinates u per tile, and points per workgroup
constexpr int kAdjStage = 32;   // coordinates v per LDS stage (two MFMA steps)
constexpr int kAdjCThreads = 256;
constexpr int kBandPts = 8;     // point blocks per band of the job order
// Four floats at any 4-byte boundary (a row of G starts at a multiple of nx).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kTabCoords = 64;  // coordinates per thread of the table kernel

struct AdjArgs {
  const float *x, *y, *z, *a;
  int64_t n;
  double pitch, wavelength;
  const float* g;
  int nx, ny, npad;
  const void *yq, *xq;
  const unsigned* gmax;
  int gblocks;
  float4* partial;
  int npb;                                      // point blocks
  int tiles_u, groups_u, slices_u, per_u, st_u;  // x part: tiles, column groups, slices,
  int tiles_p, groups_p, slices_p, per_p, st_p;  //   tiles per group, stages per slice
};

// The operands are formed from phases (two uint4 a share); else they are read.
constexpr bool forms_operands(int mode) { return mode == kHalfF16x3 || mode == kF32; }

// One part (PY: the y part) of one workgroup: point block pb, plane `plane`.
template <int MODE, bool TAB, bool PY>
__device__ __forceinline__ void adj_part(const AdjArgs& p, int pb, int plane, uint4* lds,
                                         unsigned* red) {
  constexpr bool kForms = forms_operands(MODE);
  constexpr int kPlanes = kForms ? 2 : 1;
  constexpr int kBlocks = kAdjTile / 32;
  constexpr int kBuf = 2 * kBlocks * kPlanes * kWave;  // uint4 per buffer
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int half = lane >> 5, l32 = lane & 31;
  const int sub = PY ? plane - p.groups_u * p.slices_u : plane;
  const int slices = PY ? p.slices_p : p.slices_u;
  const int per = PY ? p.per_p : p.per_u;
  const int stages_all = ((PY ? p.nx : p.ny) + kAdjStage - 1) / kAdjStage;
  const int st = PY ? p.st_p : p.st_u;
  const int slice = sub % slices, group = sub / slices;
  const int s_beg = slice * st, s_end = min(s_beg + st, stages_all);
  const int nu = PY ? p.ny : p.nx, nv = PY ? p.nx : p.ny;
  const int tile_end = min((group + 1) * per, PY ? p.tiles_p : p.tiles_u);

  const int j = pb * kAdjTile + wave * 32 + l32;   // this lane's point
  const int jc = min(j, p.npad - 1);
  const PointRecord rec = point_record(p.x, p.y, p.z, p.a, jc, p.n, p.pitch, p.wavelength);
  // Axis records of v (the contracted axis) and u (the folded one).
  const float vc = PY ? rec.xc : rec.yc, vb = PY ? rec.xb : rec.yb,
              vd = PY ? rec.xd : rec.yd;
  const float uc = PY ? rec.yc : rec.xc, ub = PY ? rec.yb : rec.xb,
              ud = PY ? rec.yd : rec.xd;
  const float pu = PY ? rec.y : rec.x;

  // Scale of G from the largest block maximum.
  unsigned m = 0;
  if (MODE != kF32) {
    for (int k = threadIdx.x; k < p.gblocks; k += kAdjCThreads) m = max(m, p.gmax[k]);
    m = group_max<kAdjCThreads>(m, red);
  }
  float mul = 1.0f, undo = 1.0f;
  if (MODE != kF32) operand_scale<MODE>(m, mul, undo);

  double d0 = 0.0, d1 = 0.0, d2 = 0.0;  // {Sc, Sx or Sy, Sr} of the blocks so far

  const char* __restrict__ vt = static_cast<const char*>(PY ? p.xq : p.yq);
  const int vquads = (nv + 3) / 4;
  // Phases of this lane's point at the eight v of step t (v = 16 t + 8 half ..).
  struct Phases {
    uint4 q0, q1;
  };
  auto load_t = [&](int t, Phases& ph) {
    if constexpr (TAB && kForms) {
      const int q = 4 * t + 2 * half;
      const char* base = vt + (int64_t)jc * 16;
      ph.q0 = *reinterpret_cast<const uint4*>(base + (int64_t)min(q, vquads - 1) * p.npad * 16);
      ph.q1 = *reinterpret_cast<const uint4*>(base + (int64_t)min(q + 1, vquads - 1) * p.npad * 16);
    } else if constexpr (TAB) {
      const int octs = (nv + 7) / 8, q = min(2 * t + half, octs - 1);
      const char* base = vt + ((int64_t)q * p.npad + jc) * 16;
      ph.q0 = *reinterpret_cast<const uint4*>(base);
      ph.q1 = *reinterpret_cast<const uint4*>(base + (int64_t)octs * p.npad * 16);
    }
  };
  auto form_t = [&](int t, const Phases& ph, Frag& C, Frag& S) {
    if constexpr (kForms) {
      float v[8];
      if constexpr (TAB) {
        const float4 a = __builtin_bit_cast(float4, ph.q0), b = __builtin_bit_cast(float4, ph.q1);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[e] = axis_phase((float)(16 * t + 8 * half + e), vc, rec.ph, rec.pl, vb, vd);
      }
      float c[8], s[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        c[e] = cos_rev(v[e]);
        s[e] = sin_rev(v[e]);
      }
      C = make_frag<MODE, true>(c);
      S = make_frag<MODE, true>(s);
    } else {
      C = Frag{ph.q0, ph.q0};
      S = Frag{ph.q1, ph.q1};
    }
  };

  for (int tile = group * per; tile < tile_end; ++tile) {
    const int u0 = tile * kAdjTile;
    floatx16 acc[kBlocks][2];
#pragma unroll
    for (int b = 0; b < kBlocks; ++b)
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][k][r] = 0.0f;

    // G: item k of a thread is eight v of one u.  In the x part a wave reads 64
    // consecutive u of a row, so the row is uniform and its address scalar; in
    // the y part four threads read the 32 v of one row.  Addresses are clamped
    // to the hologram, and what lies outside becomes zero.
    float gv[2][8];
    const int g_oct = PY ? (int)(threadIdx.x & 3) : wave >> 1;
    const int g_u = PY ? (int)(threadIdx.x >> 2) : (wave & 1) * kWave + lane;
    const float mul_u[2] = {u0 + g_u < nu ? mul : 0.0f,
                            u0 + g_u + (PY ? 64 : 0) < nu ? mul : 0.0f};
    const unsigned col = (unsigned)min(u0 + g_u, nu - 1);  // x part
    const float* __restrict__ grow[2] = {
        p.g + (PY ? (int64_t)min(u0 + g_u, nu - 1) * p.nx : 0),
        p.g + (PY ? (int64_t)min(u0 + g_u + 64, nu - 1) * p.nx : 0)};
    auto load_g = [&](int s, int k) {
      const int v0 = min(s, s_end - 1) * kAdjStage;
      if constexpr (!PY) {
        const int vv = min(v0 + 8 * (g_oct + 2 * k), nv - 1), more = nv - 1 - vv;
        const float* base = p.g + (int64_t)vv * p.nx;
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[k][e] = (base + (int64_t)min(e, more) * p.nx)[col];
      } else {
        const int vv = v0 + 8 * g_oct;
        if (v0 + kAdjStage <= nv) {
          const f32x4u a = *reinterpret_cast<const f32x4u*>(grow[k] + vv);
          const f32x4u b = *reinterpret_cast<const f32x4u*>(grow[k] + vv + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            gv[k][e] = a[e];
            gv[k][4 + e] = b[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) gv[k][e] = grow[k][min(vv + e, nv - 1)];
        }
      }
    };
    auto store_g = [&](int s, int k) {
      const int oct = g_oct + (PY ? 0 : 2 * k), u = g_u + (PY ? 64 * k : 0);
      const int vv = s * kAdjStage + 8 * oct;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // A select keeps an infinity or NaN at the edge out of the padding.  (f16x3
        // sums a G that holds one term by term; FP32 has no scale, mul is 1.)
        if constexpr (MODE == kHalfF16x3)
          v[e] = gv[k][e] * (vv + e < nv ? mul_u[k] : 0.0f);
        else
          v[e] = mul_u[k] != 0.0f && vv + e < nv ? gv[k][e] * mul : 0.0f;
      }
      const Frag f = make_frag<MODE>(v);
      uint4* d = lds + (s & 1) * kBuf + ((oct >> 1) * kBlocks + (u >> 5)) * kPlanes * kWave +
                 (oct & 1) * 32 + ((u & 31) ^ (oct * 4));
      d[0] = f.hi;
      if (kForms) d[kWave] = f.lo;
    };
    auto read_g = [&](int s, int step, int b) -> Frag {
      const uint4* q = lds + (s & 1) * kBuf + (step * kBlocks + b) * kPlanes * kWave + half * 32 +
                       (l32 ^ ((step * 2 + half) * 4));
      Frag f;
      f.hi = q[0];
      f.lo = kForms ? q[kWave] : f.hi;
      return f;
    };

    Phases ph[2];
    Frag C[2], S[2];
    const int t_last = 2 * s_end - 1;
    load_t(2 * s_beg, ph[0]);
    load_t(2 * s_beg + 1, ph[1]);
    load_g(s_beg, 0);
    load_g(s_beg, 1);
    __syncthreads();  // the buffers' last readers (the previous tile) are done
    store_g(s_beg, 0);
    store_g(s_beg, 1);
    load_g(s_beg + 1, 0);
    load_g(s_beg + 1, 1);
    form_t(2 * s_beg, ph[0], C[0], S[0]);
    load_t(min(2 * s_beg + 2, t_last), ph[0]);
    __syncthreads();
    for (int s = s_beg; s < s_end; ++s) {
      Frag A = read_g(s, 0, 0);
#pragma unroll
      for (int step = 0; step < 2; ++step) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
          const int nb = step * kBlocks + b + 1;
          const Frag next = nb < 2 * kBlocks ? read_g(s, nb / kBlocks, nb % kBlocks) : A;
          if constexpr (MODE == kF32) {
            auto part = [&](auto k) {
              acc[b][0] = mfma_part<MODE, decltype(k)::value>(A, C[step], acc[b][0]);
              acc[b][1] = mfma_part<MODE, decltype(k)::value>(A, S[step], acc[b][1]);
            };
            parts(part, std::make_integer_sequence<int, mfmas_per_step(MODE)>{});
          } else {
#pragma unroll
            for (int k = 0; k < mfmas_per_step(MODE); ++k) {
              acc[b][0] = mfma16<MODE>(k == 2 ? A.lo : A.hi, k == 1 ? C[step].lo : C[step].hi,
                                       acc[b][0]);
              acc[b][1] = mfma16<MODE>(k == 2 ? A.lo : A.hi, k == 1 ? S[step].lo : S[step].hi,
                                       acc[b][1]);
            }
          }
          A = next;
        }
        const int v = 1 - step;
        const int t = 2 * s + step;
        form_t(min(t + 1, t_last), ph[v], C[v], S[v]);
        load_t(min(t + 3, t_last), ph[v]);
        store_g(s + 1, step);
        __builtin_amdgcn_sched_barrier(0);
        load_g(s + 2, step);
      }
      __syncthreads();
    }

    // Fold over the tile's u: this lane's point, u = u0 + 32 b + 8 q + 4 half + e.
    const char* __restrict__ ut = static_cast<const char*>(PY ? p.yq : p.xq);
    const int uquads = (nu + 3) / 4;
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // FP32 within a quad, FP64 beyond.
        float s0 = 0.f, s1 = 0.f, s2 = 0.f;
        const int ub0 = u0 + 32 * b + 8 * q + 4 * half;
        float f[4];
        if constexpr (TAB && kForms) {
          const float4 t = *reinterpret_cast<const float4*>(
              ut + ((int64_t)min(ub0 / 4, uquads - 1) * p.npad + jc) * 16);
          f[0] = t.x; f[1] = t.y; f[2] = t.z; f[3] = t.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            f[e] = axis_phase((float)(ub0 + e), uc, rec.ph, rec.pl, ub, ud);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // (beyond the hologram G, and so U and V, are zero)
          const float U = acc[b][0][q * 4 + e], V = acc[b][1][q * 4 + e];
          const float c = cos_rev(f[e]), s = sin_rev(f[e]);
          const float d = (float)(ub0 + e) - pu;
          s0 = __builtin_fmaf(c, U, s0);
          s0 = __builtin_fmaf(-s, V, s0);
          const float w = __builtin_fmaf(s, U, c * V);
          s1 = __builtin_fmaf(d, w, s1);
          s2 = __builtin_fmaf(d * d, w, s2);
        }
        d0 += (double)s0;
        d1 += (double)s1;
        d2 += (double)s2;
      }
    }
  }

  float s0 = undo * (float)(d0 + __shfl_xor(d0, 32, 64));
  float s1 = undo * (float)(d1 + __shfl_xor(d1, 32, 64));
  float s2 = undo * (float)(d2 + __shfl_xor(d2, 32, 64));

  // An infinite G has no scale: such a call sums term by term (in the x part's
  // workgroups; the y part's planes are zero), so that its infinities and NaNs are the
  // direct sum's.  A NaN makes every sum NaN.
  if (MODE == kHalfF16x3 && !finite_bits(m)) {
    s0 = s1 = s2 = nan_bits(m) ? __builtin_nanf("") : 0.0f;
    float sy = s0;
    if (!PY && !nan_bits(m)) {
      for (int v = s_beg * kAdjStage; v < min(s_end * kAdjStage, nv); ++v) {
        const float Y = axis_phase((float)v, vc, rec.ph, rec.pl, vb, vd);
        const float dy = (float)v - rec.y;
        for (int u = group * per * kAdjTile + half; u < min(tile_end * kAdjTile, nu); u += 2) {
          const float t = axis_phase((float)u, uc, rec.ph, rec.pl, ub, ud) + Y;
          const float G = p.g[(int64_t)v * p.nx + u], gs = G * sin_rev(t);
          const float dx = (float)u - rec.x;
          s0 = __builtin_fmaf(G, cos_rev(t), s0);
          s1 = __builtin_fmaf(gs, dx, s1);
          sy = __builtin_fmaf(gs, dy, sy);
          s2 = __builtin_fmaf(gs, dx * dx + dy * dy, s2);
        }
      }
      s0 += __shfl_xor(s0, 32, 64);
      s1 += __shfl_xor(s1, 32, 64);
      s2 += __shfl_xor(s2, 32, 64);
      sy += __shfl_xor(sy, 32, 64);
    }
    if (half == 0 && j < p.npad) p.partial[(int64_t)plane * p.npad + j] = make_float4(s0, s1, sy, s2);
    return;
  }
  if (half == 0 && j < p.npad)
    p.partial[(int64_t)plane * p.npad + j] =
        PY ? make_float4(0.f, 0.f, s1, s2) : make_float4(s0, s1, 0.f, s2);
}

template <int MODE, bool TAB>
__global__ __launch_bounds__(kAdjCThreads, 2) void contract_adj_kernel(AdjArgs p) {
  constexpr int kPlanes = forms_operands(MODE) ? 2 : 1;
  __shared__ uint4 lds[2 * 2 * (kAdjTile / 32) * kPlanes * kWave];
  __shared__ unsigned red[kAdjCThreads / kWave];
  // Bands of kBandPts point blocks, each walked plane by plane: the workgroups
  // that run together on an XCD are then about 8 point blocks by 8 planes, and
  // share both the blocks' tables and the planes' parts of G in its L2.
  const unsigned job = xcd_tile(blockIdx.x, gridDim.x);
  const unsigned planes = gridDim.x / (unsigned)p.npb;
  const unsigned band = job / (kBandPts * planes), in_band = job - band * kBandPts * planes;
  const unsigned bh = min((unsigned)kBandPts, (unsigned)p.npb - band * kBandPts);
  const int pb = (int)(band * kBandPts + in_band % bh), plane = (int)(in_band / bh);
  if (plane >= p.groups_u * p.slices_u)
    adj_part<MODE, TAB, true>(p, pb, plane, lds, red);
  else
    adj_part<MODE, TAB, false>(p, pb, plane, lds, red);
}

// Few points or a small hologram, without tables or max |G|: a workgroup is 32
// points by tiles of 32 coordinates u, over all v.  Its eight waves take the
// steps of 16 v in turn, each forming its points' operands from their records
// and G's from memory, and add their U and V through LDS, where every thread
// then folds two (u, point) of a tile.  G is scaled by the largest |G| of the
// workgroup's own tile, which a first pass finds (the second meets it in the
// L1), so no launch before this one is needed, and short chains spread over
// the chip: 333x197, N = 700, is 22 point blocks by 18 tiles.  An operand formed
// serves 32 u here and 128 in the tiled kernel, which takes over where that
// counts.
constexpr int kDirectTile = 32;
constexpr int kDirectThreads = 512;
template <int MODE, bool PY>
__device__ __forceinline__ void direct_part(const AdjArgs& p, int pb, int plane, float* sums,
                                            unsigned* red) {
  constexpr int kWaves = kDirectThreads / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int half = lane >> 5, l32 = lane & 31;
  const int sub = PY ? plane - p.groups_u : plane, per = PY ? p.per_p : p.per_u;
  const int nu = PY ? p.ny : p.nx, nv = PY ? p.nx : p.ny;
  const int tile_end = min((sub + 1) * per, PY ? p.tiles_p : p.tiles_u);
  const int j = pb * kDirectTile + l32;  // < npad, a multiple of 64
  const PointRecord rec = point_record(p.x, p.y, p.z, p.a, j, p.n, p.pitch, p.wavelength);
  const float vc = PY ? rec.xc : rec.yc, vb = PY ? rec.xb : rec.yb,
              vd = PY ? rec.xd : rec.yd;
  const float uc = PY ? rec.yc : rec.xc, ub = PY ? rec.yb : rec.xb,
              ud = PY ? rec.yd : rec.xd;
  const float pu = PY ? rec.y : rec.x;
  const int steps = (nv + 15) / 16;
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;  // this thread's part of {Sc, Sx or Sy, Sr}

  for (int tile = sub * per; tile < tile_end; ++tile) {
    const int u0 = tile * kDirectTile;
    const bool in_u = u0 + l32 < nu;
    const int u = min(u0 + l32, nu - 1);
    // G at this lane's u and the eight v of step t, zero outside the hologram.
    auto load_g = [&](int t, float (&v)[8]) {
      const int v0 = 16 * t + 8 * half;
      if constexpr (PY) {
        const float* __restrict__ row = p.g + (int64_t)u * p.nx;
        if (v0 + 8 <= nv) {
          const f32x4u a = *reinterpret_cast<const f32x4u*>(row + v0);
          const f32x4u b = *reinterpret_cast<const f32x4u*>(row + v0 + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = in_u ? a[e] : 0.0f;
            v[4 + e] = in_u ? b[e] : 0.0f;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float g = row[min(v0 + e, nv - 1)];
            v[e] = in_u && v0 + e < nv ? g : 0.0f;
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float g = p.g[(int64_t)min(v0 + e, nv - 1) * p.nx + u];
          v[e] = in_u && v0 + e < nv ? g : 0.0f;
        }
      }
    };
    unsigned m = 0;
    float mul = 1.0f, undo = 1.0f;
    if (MODE != kF32) {
      for (int t = wave; t < steps; t += kWaves) {
        float v[8];
        load_g(t, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) m = max(m, __float_as_uint(fabsf(v[e])));
      }
      __syncthreads();  // the last tile's readers of red are done
      m = group_max<kDirectThreads>(m, red);
      operand_scale<MODE>(m, mul, undo);
    }
    // An infinite G has no scale: such a tile is summed term by term.  (A NaN makes
    // every sum NaN.)
    if (MODE == kHalfF16x3 && !finite_bits(m)) {
      float s0 = nan_bits(m) ? __builtin_nanf("") : 0.0f, s1 = s0, s2 = s0;
      for (int k = 0; k < kDirectTile && u0 + k < nu && !nan_bits(m); ++k) {
        const float U = axis_phase((float)(u0 + k), uc, rec.ph, rec.pl, ub, ud);
        const float d = (float)(u0 + k) - pu;
        for (int v = wave * 2 + half; v < nv; v += 2 * kWaves) {
          const float th = U + axis_phase((float)v, vc, rec.ph, rec.pl, vb, vd);
          const float G = p.g[PY ? (int64_t)(u0 + k) * p.nx + v : (int64_t)v * p.nx + u0 + k];
          const float gs = G * sin_rev(th);
          s0 = __builtin_fmaf(G, cos_rev(th), s0);
          s1 = __builtin_fmaf(gs, d, s1);
          s2 = __builtin_fmaf(gs, d * d, s2);
        }
      }
      d0 += (double)s0;
      d1 += (double)s1;
      d2 += (double)s2;
      continue;
    }

    floatx16 U, V;
#pragma unroll
    for (int r = 0; r < 16; ++r) U[r] = V[r] = 0.0f;
    for (int t = wave; t < steps; t += kWaves) {
      float g[8], c[8], s[8];
      load_g(t, g);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ph = axis_phase((float)(16 * t + 8 * half + e), vc, rec.ph, rec.pl, vb, vd);
        c[e] = cos_rev(ph);
        s[e] = sin_rev(ph);
        g[e] *= mul;
      }
      const Frag A = make_frag<MODE>(g), C = make_frag<MODE, true>(c), S = make_frag<MODE, true>(s);
      auto part = [&](auto k) {
        U = mfma_part<MODE, decltype(k)::value>(A, C, U);
        V = mfma_part<MODE, decltype(k)::value>(A, S, V);
      };
      parts(part, std::make_integer_sequence<int, mfmas_per_step(MODE)>{});
    }
    // Eight registers of U and of V a round: thread (w, lane) adds the waves'
    // register 8 h + w in wave order and folds it.
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        sums[((wave * 2 + 0) * 8 + k) * kWave + lane] = U[h * 8 + k];
        sums[((wave * 2 + 1) * 8 + k) * kWave + lane] = V[h * 8 + k];
      }
      __syncthreads();
      float su = sums[wave * kWave + lane], sv = sums[(8 + wave) * kWave + lane];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        su += sums[((w * 2 + 0) * 8 + wave) * kWave + lane];
        sv += sums[((w * 2 + 1) * 8 + wave) * kWave + lane];
      }
      const int r = h * 8 + wave;
      const float uu = (float)(u0 + (r >> 2) * 8 + half * 4 + (r & 3));
      const float ph = axis_phase(uu, uc, rec.ph, rec.pl, ub, ud);
      const float c = cos_rev(ph), s = sin_rev(ph), d = uu - pu;
      const float w0 = __builtin_fmaf(c, su, -(s * sv));
      const float w1 = __builtin_fmaf(s, su, c * sv);
      d0 += (double)undo * (double)w0;
      d1 += (double)undo * (double)(d * w1);
      d2 += (double)undo * (double)(d * d * w1);
    }
  }

  // The sixteen threads of a point, in order.
  d0 += __shfl_xor(d0, 32, 64);
  d1 += __shfl_xor(d1, 32, 64);
  d2 += __shfl_xor(d2, 32, 64);
  __syncthreads();
  double* all = reinterpret_cast<double*>(sums);
  if (half == 0) {
    all[(wave * 3 + 0) * 32 + l32] = d0;
    all[(wave * 3 + 1) * 32 + l32] = d1;
    all[(wave * 3 + 2) * 32 + l32] = d2;
  }
  __syncthreads();
  if (threadIdx.x < 32) {
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      d0 += all[(w * 3 + 0) * 32 + l32];
      d1 += all[(w * 3 + 1) * 32 + l32];
      d2 += all[(w * 3 + 2) * 32 + l32];
    }
    p.partial[(int64_t)plane * p.npad + j] =
        PY ? make_float4(0.f, 0.f, (float)d1, (float)d2)
           : make_float4((float)d0, (float)d1, 0.f, (float)d2);
  }
}

template <int MODE>
__global__ __launch_bounds__(kDirectThreads) void contract_adj_direct_kernel(AdjArgs p) {
  constexpr int kWaves = kDirectThreads / kWave;
  __shared__ double sums[kWaves * 16 * kWave / 2];
  __shared__ unsigned red[kWaves];
  const unsigned job = xcd_tile(blockIdx.x, gridDim.x);
  const int plane = (int)(job / (unsigned)p.npb), pb = (int)(job % (unsigned)p.npb);
  if (plane >= p.groups_u)
    direct_part<MODE, true>(p, pb, plane, reinterpret_cast<float*>(sums), red);
  else
    direct_part<MODE, false>(p, pb, plane, reinterpret_cast<float*>(sums), red);
}

// Largest |G| per workgroup (blockIdx.x < gblocks) and, in the same launch, the
// phase tables of both axes: the workgroups after those take 256 points and
// kTabCoords coordinates each (rows first), a thread its point's quads.
template <int MODE>
__global__ __launch_bounds__(256) void contract_adj_tables_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ a, int64_t n, int npad, double pitch, double wavelength,
    const float* __restrict__ g, int64_t pixels, int gblocks, unsigned* __restrict__ gmax, int ny,
    int nx, int pblocks, int yslices, uint4* __restrict__ yq, uint4* __restrict__ xq) {
  __shared__ unsigned red[4];
  if ((int)blockIdx.x < gblocks) {
    unsigned m = 0;
    auto take = [&](float v) { m = max(m, __float_as_uint(fabsf(v))); };
    const int64_t stride = (int64_t)gblocks * 256;
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int64_t done = 0;
    if (((uintptr_t)g & 15u) == 0) {
      const float4* g4 = reinterpret_cast<const float4*>(g);
      const int64_t n4 = pixels / 4;
      int64_t i = first;
      for (; i + 3 * stride < n4; i += 4 * stride) {
        float4 q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = g4[i + k * stride];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          take(q[k].x);
          take(q[k].y);
          take(q[k].z);
          take(q[k].w);
        }
      }
      for (; i < n4; i += stride) {
        const float4 q = g4[i];
        take(q.x);
        take(q.y);
        take(q.z);
        take(q.w);
      }
      done = 4 * n4;
    }
    for (int64_t i = done + first; i < pixels; i += stride) take(g[i]);
    m = group_max<256>(m, red);
    if (threadIdx.x == 0) gmax[blockIdx.x] = m;
    return;
  }
  const int b = (int)blockIdx.x - gblocks;
  const int j = (b % pblocks) * 256 + (int)threadIdx.x;
  if (j >= npad) return;
  const int slice = b / pblocks;
  const bool is_y = slice < yslices;
  const int h0 = (is_y ? slice : slice - yslices) * kTabCoords;
  const int size = is_y ? ny : nx;
  const PointRecord r = point_record(x, y, z, a, j, n, pitch, wavelength);
  const float c = is_y ? r.yc : r.xc, pb = is_y ? r.yb : r.xb, d = is_y ? r.yd : r.xd;
  uint4* dst = is_y ? yq : xq;
  auto phase = [&](int h) { return axis_phase((float)h, c, r.ph, r.pl, pb, d); };
  if constexpr (MODE == kHalfF16x3 || MODE == kF32) {
    const int quads = (size + 3) / 4;
    for (int q = h0 / 4; q < min((h0 + kTabCoords) / 4, quads); ++q)
      dst[(int64_t)q * npad + j] =
          make_uint4(__float_as_uint(phase(4 * q)), __float_as_uint(phase(4 * q + 1)),
                     __float_as_uint(phase(4 * q + 2)), __float_as_uint(phase(4 * q + 3)));
  } else {
    const int octs = (size + 7) / 8;
    for (int q = h0 / 8; q < min((h0 + kTabCoords) / 8, octs); ++q) {
      float cs[8], sn[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float ph = phase(8 * q + e);
        cs[e] = cos_rev(ph);
        sn[e] = sin_rev(ph);
      }
      dst[(int64_t)q * npad + j] = make_frag<MODE>(cs).hi;
      dst[((int64_t)octs + q) * npad + j] = make_frag<MODE>(sn).hi;
    }
  }
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Plans the direct kernel where a model of its time is below that of the tiled
// plan, which takes `best` units (none if negative).  Of the direct kernel's
// workgroups 512 run at once; each takes 3.2 us and 0.31 a step of its longer
// axis, and one alone on its CU 0.55 of that.  (us a call, tiled and direct:
// 333x197, N = 700: 24.6 and 20.6; N = 2048: 28.9 and 29.9; 256x256, N = 1024:
// 25.3 and 20.5; 1024x1024, N = 256: 29.4 and 33.2; 1920x1080, N = 128: 30.7 and
// 47.2.  Both include 20 us of the host's that hide shorter kernels.)
bool plan_direct(const Plan& p, int64_t capacity, double best, ContractAdj& c) {
  const int64_t tiles_u = ceil_div(p.nx, kDirectTile), tiles_p = ceil_div(p.ny, kDirectTile);
  const double wgs = (double)(tiles_u + tiles_p) * (double)(p.npad / kDirectTile);
  const double steps = (double)ceil_div(std::max(p.nx, p.ny), 16);
  const double direct = 9.5 + std::max(0.55, wgs / 512) * (3.2 + 0.31 * steps);
  if (best >= 0.0 && direct >= 9.0 + (c.mode == kF32 ? 4.0 : 2.0) * best) return false;
  int64_t per = 1;
  while (ceil_div(tiles_u, per) + ceil_div(tiles_p, per) > capacity && per < tiles_u + tiles_p) ++per;
  const int64_t planes = ceil_div(tiles_u, per) + ceil_div(tiles_p, per);
  if (planes > capacity || planes * (p.npad / kDirectTile) > 0x7fffffff) return false;
  c.direct = true;
  c.groups_u = (int)ceil_div(tiles_u, per);
  c.groups_p = (int)ceil_div(tiles_p, per);
  c.slices_u = c.slices_p = 1;
  c.planes = (int)planes;
  return true;
}

}  // namespace

bool plan_contract_adj(const Plan& p, const Workspace& w, ContractAdj& c) {
  c = ContractAdj{};
  if (p.op != 2) return false;
  int64_t capacity;
  if (p.variant == 1) {
    // Below 32 rows most of the 128 rows of a tile of the y part are padding,
    // and the direct adjoint is faster (1920x16, N = 1024: 27 against 35 us a
    // call; 4096x4, N = 16448: 150 against 307; at 1920x32 both take 35, at
    // 1920x64 52 against 36).
    if (p.ny < 32) return false;
    c.mode = kHalfF16x3;
    c.yq = w.rtab;
    c.xq = w.ctab;
    // The row table's region holds 8 bytes a row and point; the phase table
    // takes 4.
    c.tab = w.rtab && w.ctab;
    c.partial = (float4*)w.partial;
    capacity = p.regions;
  } else {
    c.mode = p.variant == 2 ? kF32 : p.variant == 3 ? kHalfF16x3 : p.variant == 4 ? kHalfF16 : kHalfBF16;
    c.yq = p.variant == 2 ? w.sep_y : w.htab_y;
    c.xq = p.variant == 2 ? w.sep_x : w.htab_x;
    c.tab = true;
    c.partial = w.fold;
    capacity = p.fold_planes;
  }
  c.gmax = (unsigned*)(c.partial + capacity * p.npad);
  // (the FP32 operands take no scale)
  c.gblocks = c.mode == kF32 ? 0 : (int)std::min<int64_t>(kMaxGBlocks, ceil_div((int64_t)p.nx * p.ny, 256 * 8));
  // Tiles per workgroup and slices of v.  A workgroup takes, in units of one
  // stage, kStart to begin with and for each of its tiles the slice's stages and
  // fold for the fold; 512 run at once, two a CU, and one alone on its CU takes
  // `alone` of that.  For every length t a workgroup may take, each part gets as few
  // workgroups as keep within it, and the plan with the least time is taken:
  // one workgroup's where all run at once, else the work over the slots and
  // part of a workgroup's tail.  Workgroups beyond kLongest stages drift apart and
  // lose each other's G and tables in L2 (3840x2160, N = 16384: 3.14 to 3.2 ms
  // with 75 to 342 stages, 3.5 with 1139), so they are not made longer than a
  // tile needs.  At 46 random sizes the choice is within 1% of the best on
  // average, 16% at most.  In FP32 a stage takes 2.6 times as long on the matrix
  // cores, so the fold counts for less and a workgroup alone on its CU gains
  // more (the terms below: within 1% on average, 7% at most, over 34 sizes;
  // 1449x1371, N = 1730: 333 us where the f16x3 terms' plan took 401).
  constexpr int64_t kSlots = 512, kStart = 1, kLongest = 350;
  const int64_t fold = c.mode == kF32 ? 1 : 6;
  const double alone = c.mode == kF32 ? 0.55 : 0.7, tail = c.mode == kF32 ? 0.35 : 0.5;
  const int64_t npb = ceil_div(p.npad, kAdjTile);
  const int64_t tiles[2] = {ceil_div(p.nx, kAdjTile), ceil_div(p.ny, kAdjTile)};
  const int64_t stages[2] = {ceil_div(p.ny, kAdjStage), ceil_div(p.nx, kAdjStage)};
  double best = -1.0;
  const int64_t all = kStart + std::max(tiles[0] * (stages[0] + fold), tiles[1] * (stages[1] + fold));
  const int64_t one_tile = kStart + fold + std::max(stages[0], stages[1]);
  for (int64_t t = kStart + fold + 2;; t = t + 1 + t / 16) {
    if (t > all) t = all;
    int64_t groups[2], slices[2], wgs = 0, work = 0, longest = 0;
    for (int k = 0; k < 2; ++k) {
      const int64_t one = stages[k] + fold, room = t - kStart;
      if (room >= one) {
        groups[k] = ceil_div(tiles[k], room / one);
        slices[k] = 1;
      } else {
        groups[k] = tiles[k];
        slices[k] = ceil_div(stages[k], room - fold);
        slices[k] = ceil_div(stages[k], ceil_div(stages[k], slices[k]));  // none empty
      }
      wgs += groups[k] * slices[k];
      work += groups[k] * slices[k] * kStart + tiles[k] * (stages[k] + fold * slices[k]);
      longest = std::max(longest, kStart + ceil_div(tiles[k], groups[k]) *
                                               (ceil_div(stages[k], slices[k]) + fold));
    }
    if (wgs <= capacity) {
      const int64_t n = wgs * npb;
      const double time = n <= kSlots / 2 ? alone * longest
                          : n <= kSlots   ? (double)longest
                                          : std::max((double)longest, (double)(work * npb) / kSlots +
                                                                          tail * longest);
      if (best < 0.0 || time < best) {
        best = time;
        c.groups_u = (int)groups[0];
        c.slices_u = (int)slices[0];
        c.groups_p = (int)groups[1];
        c.slices_p = (int)slices[1];
      }
    }
    if (t == all || (best >= 0.0 && t > std::max(one_tile, kLongest))) break;
  }
  if (plan_direct(p, capacity, best, c)) return true;
  if (best < 0.0) return false;
  c.planes = c.groups_u * c.slices_u + c.groups_p * c.slices_p;
  return c.planes * npb <= 0x7fffffff;
}

hipError_t launch_contract_adj_tables(const Plan& p, const ContractAdj& c, const float* x,
                                      const float* y, const float* z, const float* a,
                                      double pitch, double wavelength, const float* g,
                                      hipStream_t s) {
  const int pblocks = (int)ceil_div(p.npad, 256);
  const int yslices = c.tab ? (int)ceil_div(p.ny, kTabCoords) : 0;
  const int xslices = c.tab ? (int)ceil_div(p.nx, kTabCoords) : 0;
  const int64_t blocks = c.gblocks + (int64_t)pblocks * (yslices + xslices);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, y, z, a, p.n,
                       (int)p.npad, pitch, wavelength, g, (int64_t)p.nx * p.ny, c.gblocks, c.gmax,
                       p.ny, p.nx, pblocks, yslices, (uint4*)c.yq, (uint4*)c.xq);
  };
  if (c.mode == kHalfF16x3 || c.mode == kF32)
    go(contract_adj_tables_kernel<kHalfF16x3>);
  else if (c.mode == kHalfF16)
    go(contract_adj_tables_kernel<kHalfF16>);
  else
    go(contract_adj_tables_kernel<kHalfBF16>);
  return hipGetLastError();
}

hipError_t launch_contract_adj(const Plan& p, const ContractAdj& c, const float* x,
                               const float* y, const float* z, const float* a, double pitch,
                               double wavelength, const float* g, hipStream_t s) {
  AdjArgs r{};
  r.x = x;
  r.y = y;
  r.z = z;
  r.a = a;
  r.n = p.n;
  r.pitch = pitch;
  r.wavelength = wavelength;
  r.g = g;
  r.nx = p.nx;
  r.ny = p.ny;
  r.npad = (int)p.npad;
  r.yq = c.yq;
  r.xq = c.xq;
  r.gmax = c.gmax;
  r.gblocks = c.gblocks;
  r.partial = c.partial;
  const int tile = c.direct ? kDirectTile : kAdjTile;
  r.npb = (int)ceil_div(p.npad, tile);
  r.tiles_u = (int)ceil_div(p.nx, tile);
  r.groups_u = c.groups_u;
  r.slices_u = c.slices_u;
  r.per_u = (int)ceil_div(r.tiles_u, c.groups_u);
  r.st_u = (int)ceil_div(ceil_div(p.ny, kAdjStage), c.slices_u);
  r.tiles_p = (int)ceil_div(p.ny, tile);
  r.groups_p = c.groups_p;
  r.slices_p = c.slices_p;
  r.per_p = (int)ceil_div(r.tiles_p, c.groups_p);
  r.st_p = (int)ceil_div(ceil_div(p.nx, kAdjStage), c.slices_p);
  const dim3 grid((unsigned)(r.npb * c.planes)), block(c.direct ? kDirectThreads : kAdjCThreads);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, r); };
  if (c.direct && c.mode == kHalfF16x3)
    go(contract_adj_direct_kernel<kHalfF16x3>);
  else if (c.direct && c.mode == kF32)
    go(contract_adj_direct_kernel<kF32>);
  else if (c.direct && c.mode == kHalfF16)
    go(contract_adj_direct_kernel<kHalfF16>);
  else if (c.direct)
    go(contract_adj_direct_kernel<kHalfBF16>);
  else if (c.mode == kHalfF16x3 && c.tab)
    go(contract_adj_kernel<kHalfF16x3, true>);
  else if (c.mode == kHalfF16x3)
    go(contract_adj_kernel<kHalfF16x3, false>);
  else if (c.mode == kF32)
    go(contract_adj_kernel<kF32, true>);
  else if (c.mode == kHalfF16)
    go(contract_adj_kernel<kHalfF16, true>);
  else
    go(contract_adj_kernel<kHalfBF16, true>);
  return hipGetLastError();
}

}  // namespace cgh
