// The hologram sum and its adjoint as contractions on the matrix cores,
// with the operands formed inside the kernels (contract_fwd.hip,
// contract_adj.hip).
//
// The phase of Eq. (1) (Section 1) separates by axis, theta = X_j(x) + Y_j(y)
// revolutions, each part the compensated axis_phase, and by the addition
// theorem cos(X + Y) = cX cY - sX sY, so the sum over points is a contraction
// of per-axis cosines and sines.  A value v enters the matrix cores in one of
// these formats (FP32 accumulation in all):
//
//   kHalfF16x3  v = hi + lo, hi = fp16(v), lo = fp16(v - hi), three products
//               hi*hi + hi*lo + lo*hi: the planes are off by 2^-23 |v| at most or,
//               as lo's smallest step is 2^-24, by 2^-25 where that is more (|v|
//               below 1/4: a small cosine has fewer bits of its own, 20 at 1/32),
//               and what is dropped, lo*lo, is below 2^-22 of the product.
//   kHalfF16, kHalfBF16   v rounded once to 16 bits, one product.
//   kF32        v itself, on the FP32 matrix cores.
//
// Cosines and sines lie in [-1, 1].  The other operand's values (A_j forward, G
// in the adjoint) are multiplied by a power of two first (exact), which puts the
// largest below 2^15 (f16x3) or 1 (the single planes): with fp16's smallest step
// at 2^-24, a value down to 2^-16 of the largest keeps both planes at full width,
// and the absolute error of a smaller one is below 2^-39 of the largest.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "cgh_internal.h"
#include "order.h"
#include "phase.h"

namespace cgh {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One lane's share of a 32 x 16 operand block of v_mfma_f32_32x32x16: row (or
// column) lane % 32, k = (lane / 32) * 8 .. + 7, two 16-bit values a dword (kF32:
// the eight values themselves).
struct Frag {
  uint4 hi, lo;
};

template <int MODE>
__device__ __forceinline__ floatx16 mfma16(uint4 a, uint4 b, floatx16 c) {
  if constexpr (MODE == kHalfBF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a),
                                                  __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
}

// acc += A B over one step (k = 16): the planes' products, or for kF32 eight
// v_mfma_f32_32x32x2, the t-th with every lane's t-th value (its k is then (lane
// / 32) * 8 + t on both sides).
template <class F, int... K>
__device__ __forceinline__ void parts(F&& f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);  // for each k of the sequence
}
constexpr int mfmas_per_step(int mode) {
  return mode == kF32 ? 8 : mode == kHalfF16x3 ? 3 : 1;
}
template <int MODE, int K>
__device__ __forceinline__ floatx16 mfma_part(const Frag& a, const Frag& b, floatx16 c) {
  if constexpr (MODE == kF32) {
    const uint32_t va[8] = {a.hi.x, a.hi.y, a.hi.z, a.hi.w, a.lo.x, a.lo.y, a.lo.z, a.lo.w};
    const uint32_t vb[8] = {b.hi.x, b.hi.y, b.hi.z, b.hi.w, b.lo.x, b.lo.y, b.lo.z, b.lo.w};
    return __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(va[K]), __uint_as_float(vb[K]), c,
                                                0, 0, 0);
  } else {
    return mfma16<MODE>(K == 2 ? a.lo : a.hi, K == 1 ? b.lo : b.hi, c);
  }
}

// Two values rounded to the 16-bit format (to nearest even), v0 in the low half.
template <int MODE>
__device__ __forceinline__ uint32_t pack16(float v0, float v1) {
  if constexpr (MODE == kHalfBF16) {
    const bf16x2 h = {(__bf16)v0, (__bf16)v1};
    return __builtin_bit_cast(uint32_t, h);
  } else {
    const halfx2 h = {(_Float16)v0, (_Float16)v1};
    return __builtin_bit_cast(uint32_t, h);
  }
}

// hi and lo planes of two values: v_cvt_pk_f16_f32, two v_fma_mix_f32 for the
// differences v - hi (exact) and another pack.  The two empty asm statements
// keep the compiler from converting each value a second time for the
// difference and from turning the fma into a conversion and a subtraction.
// With RAISE the planes hold v (1 + 2^-24) instead, an empirical gain: the native
// cosine and sine are 3.3e-8 too small on average (measured as the scale of a
// hologram), so a product of two is 6.6e-8 too small, which one raised operand takes
// back.  It is in lo, so it is exact for the scaled operand that the forward raises
// (scale -6.6e-8 without, -0.9e-8 with); of the cosines and sines that the adjoint
// raises, near lo's smallest step, 0.7 to 1.04 of it arrives by octave of v.
template <bool RAISE>
__device__ __forceinline__ void split16(float v0, float v1, uint32_t& hi, uint32_t& lo) {
  uint32_t h = pack16<kHalfF16x3>(v0, v1);
  float neg = RAISE ? -0x1.fffffep-1f : -1.0f;
  asm("" : "+v"(h));
  asm("" : "+v"(neg));
  const halfx2 hh = __builtin_bit_cast(halfx2, h);
  hi = h;
  lo = pack16<kHalfF16x3>(__builtin_fmaf((float)hh[0], neg, v0),
                          __builtin_fmaf((float)hh[1], neg, v1));
}

// Eight values as one lane's share of a block (k in order).
template <int MODE, bool RAISE = false>
__device__ __forceinline__ Frag make_frag(const float (&v)[8]) {
  Frag f;
  if constexpr (MODE == kF32) {
    f.hi = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                      __float_as_uint(v[3]));
    f.lo = make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]),
                      __float_as_uint(v[7]));
  } else if constexpr (MODE == kHalfF16x3) {
    split16<RAISE>(v[0], v[1], f.hi.x, f.lo.x);
    split16<RAISE>(v[2], v[3], f.hi.y, f.lo.y);
    split16<RAISE>(v[4], v[5], f.hi.z, f.lo.z);
    split16<RAISE>(v[6], v[7], f.hi.w, f.lo.w);
  } else {
    f.hi = make_uint4(pack16<MODE>(v[0], v[1]), pack16<MODE>(v[2], v[3]),
                      pack16<MODE>(v[4], v[5]), pack16<MODE>(v[6], v[7]));
    f.lo = make_uint4(0, 0, 0, 0);
  }
  return f;
}

// The power of two that an operand with the largest magnitude m (its float bits; 1
// where m is 0 or not finite) is multiplied by, and its inverse.  frexp's exponent e (m < 2^e)
// is clamped so that both stay normal floats.  The largest value is then below 2^TOP.
template <int MODE, int TOP = MODE == kHalfF16x3 ? 15 : 0>
__device__ __forceinline__ void operand_scale(unsigned max_bits, float& mul, float& undo) {
  int e = 0;
  const float m = __uint_as_float(max_bits);
  if (m > 0.0f && m < __builtin_inff()) {
    (void)frexpf(m, &e);
    e -= TOP;
  }
  e = max(-126, min(126, e));
  undo = ldexpf(1.0f, e);
  mul = ldexpf(1.0f, -e);
}
__device__ __forceinline__ bool finite_bits(unsigned max_bits) { return max_bits < 0x7f800000u; }
__device__ __forceinline__ bool nan_bits(unsigned max_bits) { return max_bits > 0x7f800000u; }

// Largest of v over a workgroup of T threads, on every thread; `lds` holds one
// word per wave.  (Non-negative floats order as their bits.)
template <int T>
__device__ __forceinline__ unsigned group_max(unsigned v, unsigned* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, 64));
  if constexpr (T > kWave) {
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    v = lds[0];
#pragma unroll
    for (int w = 1; w < T / kWave; ++w) v = max(v, lds[w]);
    __syncthreads();
  }
  return v;
}

// ----------------------------------------------------------------- forward --
// Tables of the forward, a quad of points at a time so that a lane's four
// points of one coordinate are one 16-byte load and 32 lanes of consecutive
// coordinates read 512 consecutive bytes:
//   f16x3        float [npad / 4][rows][4]   the axis phase
//   f32          two planes float [npad / 4][rows][4]: (cos, sin) of the quad's
//                first two points, of its other two
//   f16, bf16    uint32 [npad / 4][rows][4]  (cos, sin) as two 16-bit values
// y rows (with A_j and the scale in the 16-bit values), then x columns.
struct FwdOperands {
  const void* yq;     // [npad / 4][rows_y][4]
  const void* xq;     // [npad / 4][cols_x][4], or null: from the records
  const float4* rec;  // [npad / 4][5] x records {c, ph, pl, b, d} by quad, when xq is null
  const float* amp;   // [npad]
  int rows_y, cols_x;
};

constexpr int kOrdered = 6;  // the shape whose slices are sums of their points in order
struct ContractFwd {
  int mode;           // the operand format
  bool direct;        // one launch without tables (few points), else:
  int shape;          // index of the kernel's tile shape
  int rows_y, cols_x;
  bool xtab;
  void* yq;
  void* xq;
  float4* rec;
  float* amp;
  unsigned* amax;     // [kWave] maxima of |A| as float bits (single planes, kOrdered)
  int64_t chunk;      // points per pass where the tables of all have no room (else 0)
  int slices;         // the points are cut into this many slices,
  float* planes;      //   with a plane [ny][nx] each when there are several
};
bool plan_contract_fwd(const Plan& p, const Workspace& w, ContractFwd& c);
// The number of point slices of the f16x3 forward given room for any number.
int contract_fwd_slices(int64_t npad, int32_t nx, int32_t ny);
hipError_t launch_contract_fwd_tables(const Plan& p, const ContractFwd& c, const float* x,
                                      const float* y, const float* z, const float* a,
                                      double pitch, double wavelength, hipStream_t s);
// The chunks of points one after the other, each with its tables and its sum, which
// is added to the ones before.
hipError_t launch_contract_chunks(const Plan& p, const ContractFwd& c, const float* x,
                                  const float* y, const float* z, const float* a, double pitch,
                                  double wavelength, float* out, const float* target,
                                  float* residual, hipStream_t s);
hipError_t launch_contract_direct(const Plan& p, const ContractFwd& c, const float* x,
                                  const float* y, const float* z, const float* a, double pitch,
                                  double wavelength, float* out, const float* target,
                                  float* residual, hipStream_t s);
hipError_t launch_contract_fwd(const Plan& p, const ContractFwd& c, float* out,
                               const float* target, float* residual, hipStream_t s);

// -------------------------------------------------------------- FP64 forward --
// Bytes of tables that a chunk of points may take (16 a point and coordinate):
// large enough that a chunk's launches and its pass over the hologram are small
// beside its products (3840x2160: 1344 points a chunk, about 0.6 ms).
constexpr int64_t kF64TableBytes = int64_t(128) << 20;
void plan_contract_f64(Plan& p);  // sets f64_chunk and f64_slices
size_t contract_f64_table_bytes(const Plan& p);
hipError_t launch_contract_f64(const Plan& p, const Workspace& w, const float* x, const float* y,
                               const float* z, const float* a, double pitch, double wavelength,
                               double* out, hipStream_t s);

// ----------------------------------------------------------------- adjoint --
// Tables of the adjoint, a quad of coordinates at a time (lane = point):
//   f16x3, f32   float [ceil(size / 4)][npad][4]   the axis phase
//   f16, bf16    two planes uint32 [ceil(size / 8)][npad][4]: cosines, sines
constexpr int kMaxGBlocks = 512;  // block maxima of |G|, behind the partial planes
struct ContractAdj {
  int mode;
  bool direct;        // no tables: the points' records and 32-wide tiles
  bool tab;           // the tables exist (else the kernel forms the phases)
  void *yq, *xq;
  unsigned* gmax;     // [gblocks] block maxima of |G| (float bits)
  int gblocks;
  float4* partial;    // [planes][npad] {Sc, Sx, Sy, Sr}
  int planes;
  int groups_u, slices_u, groups_p, slices_p;  // column groups x K slices of each part
};
bool plan_contract_adj(const Plan& p, const Workspace& w, ContractAdj& c);
hipError_t launch_contract_adj_tables(const Plan& p, const ContractAdj& c, const float* x,
                                      const float* y, const float* z, const float* a,
                                      double pitch, double wavelength, const float* g,
                                      hipStream_t s);
hipError_t launch_contract_adj(const Plan& p, const ContractAdj& c, const float* x,
                               const float* y, const float* z, const float* a, double pitch,
                               double wavelength, const float* g, hipStream_t s);

}  // namespace cgh
