// Device helpers that the kernels working on chart rows share: reductions, operand planes, exponents of the scaled
// representation (see spcfg_internal.h), the row of a span.
#pragma once
#include "gemm_nt_common.h"

namespace spcfg {

namespace {

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block-wide reductions through LDS; `red` needs one slot per wave (<= 16). All threads get the result.
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max(v);
  const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  float r = red[0];
  for (int i = 1; i < nw; ++i) r = fmaxf(r, red[i]);
  return r;
}
__device__ __forceinline__ int block_max_i(int v, int* red) {
  v = wave_max_i(v);
  const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  int r = red[0];
  for (int i = 1; i < nw; ++i) r = max(r, red[i]);
  return r;
}
__device__ __forceinline__ double block_sum_d(double v, double* red) {
  v = wave_sum_d(v);
  const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < nw; ++i) r += red[i];
  return r;
}

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
// bf16 copy of four consecutive values (round to nearest even): the operand the bf16 projection products read
__device__ __forceinline__ void store_bf16x4(void* base, int64_t idx, float4 v) {
  bf16x4_t r;
  r[0] = (__bf16)v.x; r[1] = (__bf16)v.y; r[2] = (__bf16)v.z; r[3] = (__bf16)v.w;
  *reinterpret_cast<bf16x4_t*>(static_cast<__bf16*>(base) + idx) = r;
}

// Operand planes of four consecutive values for the projection products: with three planes the exact cut
// x = hi + mid + lo into bf16 pieces (nt::Split3), with two planes hi = bf16(x) and lo = bf16(x - hi) (the first two
// pieces of the same cut), with one plane the bf16 rounding.  Plane p starts at base + p * plane_stride elements.
__device__ __forceinline__ void store_planes4(void* base, int planes, int64_t plane_stride, int64_t idx, float4 v) {
  if (planes >= 2) {
    unsigned h0, m0, l0, h1, m1, l1;
    nt::Split3::cut2(v.x, v.y, h0, m0, l0);
    nt::Split3::cut2(v.z, v.w, h1, m1, l1);
    uint16_t* b = static_cast<uint16_t*>(base) + idx;
    *reinterpret_cast<uint2*>(b) = uint2{h0, h1};
    *reinterpret_cast<uint2*>(b + plane_stride) = uint2{m0, m1};
    if (planes == 3) *reinterpret_cast<uint2*>(b + 2 * plane_stride) = uint2{l0, l1};
  } else {
    store_bf16x4(base, idx, v);
  }
}

// 2^d as a float for an integer d (0 below the fp32 range); exact.
__device__ __forceinline__ float pow2i(int d) { return d < -160 ? 0.0f : ldexpf(1.0f, min(d, 127)); }

__device__ __forceinline__ int add_exp(int a, int b) { return (a == kExpZero || b == kExpZero) ? kExpZero : a + b; }

// A stored vector has a raw exponent m and the bit pattern of its largest magnitude (kept by integer
// atomicMax, which is exact and order-independent).  Its normalising shift f puts that maximum into
// [0.5, 1): the vector's consumers use the exponent m + f and the scale 2^-f.
__device__ __forceinline__ int norm_shift(uint32_t maxbits) { return max((int)((maxbits >> 23) & 0xffu) - 126, -126); }
__device__ __forceinline__ int norm_exp(int m, uint32_t maxbits) {
  return (maxbits == 0u || m == kExpZero) ? kExpZero : m + norm_shift(maxbits);
}
__device__ __forceinline__ float norm_scale(uint32_t maxbits) {
  return maxbits == 0u ? 0.0f : ldexpf(1.0f, -norm_shift(maxbits));
}

// A projected half row (eta or zeta of a span) is stored as 2^-f * [L or R] * (stored inside vector), with the
// exponent m + f of its inside vector (f = norm_shift(tmaxb)).  Its producer also records
//   psum = max_B (biased exponent of max_A W[A,B]) + (biased exponent of the stored inside entry B)      (0: all zero)
// so that the largest entry of W * (stored inside vector) lies in [2^(psum - 254), 4 N 2^(psum - 254)).  The
// consumers read the half row as 2^-g * stored with g = (psum - 253) - f (clamped to the fp32 exponent range): its
// largest entry is then in [0.5, 2 N), and products of two such values cannot leave the fp32 range however small
// (or large) the grammar's weights are.
__device__ __forceinline__ int bexp(float x) { return (int)((__float_as_uint(x) >> 23) & 0xffu); }
__device__ __forceinline__ int bexp_sum(float w, float x) {
  const int a = bexp(w), b = bexp(x);
  return (a == 0 || b == 0) ? 0 : a + b;
}
__device__ __forceinline__ int proj_shift(uint32_t tmaxbits, int psum) {
  return min(max((psum - 253) - norm_shift(tmaxbits), -126), 126);
}
__device__ __forceinline__ int proj_exp(int m, uint32_t tmaxbits, int psum) {
  const int e = norm_exp(m, tmaxbits);
  return (e == kExpZero || psum == 0) ? kExpZero : e + proj_shift(tmaxbits, psum);
}

// Row of span (i, i + w) of sentence b of length n (rowtab: see the span plan in kernels_elem.hip)
__device__ __forceinline__ int row_of(const int32_t* __restrict__ rowtab, int stride, int B, int w, int b, int i,
                                      int n) {
  const int which = i == 0 ? 0 : (i == n - w ? 2 : 1);
  return rowtab[which * stride + w * B + b] + (which == 1 ? i - 1 : 0);
}

// Where the exponents of row r's partial sums of the reverse pass lie (which: 0 adjoint of eta, 1 of zeta): in the row's place
// of BH until its reverse product, for leaf rows in two arrays that the reverse pass does not read.
struct BwdPartExp {
  float* BH;
  float* xs;
  int32_t* rootmask;
  __device__ __forceinline__ void put(int which, int64_t r, int64_t S1, int Np, int32_t e) const {
    if (r >= S1) BH[(r - S1) * Np + which] = __int_as_float(e);
    else if (which == 0) xs[r] = __int_as_float(e);
    else rootmask[r] = e;
  }
};
// (through the launches' own pointers: where the row is the same for a wavefront, as in the kernels of one width, a uniform load that
// goes through the scalar cache)
__device__ __forceinline__ int2 bwd_part_exp(int w, int64_t r, int64_t S1, int Np, const float* __restrict__ BH,
                                             const float* __restrict__ xs, const int32_t* __restrict__ rootmask) {
  if (w == 1) return make_int2(__float_as_int(xs[r]), rootmask[r]);
  return make_int2(__float_as_int(BH[(r - S1) * Np]), __float_as_int(BH[(r - S1) * Np + 1]));
}

}  // namespace

}  // namespace spcfg
