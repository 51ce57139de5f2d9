// Device functions shared by the streaming kernels over FP32 operands (fused.hip, strips.hip).
#ifndef SRQ_STREAM_H_
#define SRQ_STREAM_H_
#include "srq_internal.h"

namespace srq {

static __device__ __forceinline__ float block_max_256(float m, float* sm) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  __syncthreads();                                   // sm may still be read from a previous use
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
  __syncthreads();
  return fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
}

// Four floats or packed codes at any address their element allows: the target takes unaligned vector
// accesses, so a row of any length and leading dimension is read with the same 16-byte loads as an
// aligned one (where a piece straddles two lines it costs a second one, which the next lane asks for
// anyway).
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u1u __attribute__((aligned(1)));
typedef unsigned u4u __attribute__((ext_vector_type(4), aligned(1)));

// 16-byte load that does not displace cached data (used for the last read of an operand before
// a product runs in between)
static __device__ __forceinline__ float4 load_streaming(const float* p) {
  const f4u t = __builtin_nontemporal_load(reinterpret_cast<const f4u*>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}

// the first n (0..4) of the four values at p, zero for the others
static __device__ __forceinline__ float4 load_part(const float* p, int n) {
  if (n >= 4) {
    const f4u t = *reinterpret_cast<const f4u*>(p);
    return make_float4(t.x, t.y, t.z, t.w);
  }
  return make_float4(n > 0 ? p[0] : 0.f, n > 1 ? p[1] : 0.f, n > 2 ? p[2] : 0.f, 0.f);
}

// The same without a branch, for rows of `len` (at least 4) values: the values at .. at + 3 of a row, zero from len on, in two
// steps, so that many loads can be on their way together (a load behind a branch is waited for before the next
// is issued): a load from a place that exists, and the shift to where it was wanted.
static __device__ __forceinline__ f4u load_inside(const float* row, int at, int len) {
  return *reinterpret_cast<const f4u*>(row + (at < len - 4 ? at : len - 4));
}
static __device__ __forceinline__ float4 shifted(f4u x, int at, int len) {
  const int past = at - (len - 4);                   // <= 0: the load was where it was wanted
  if (past <= 0) return make_float4(x.x, x.y, x.z, x.w);
  return make_float4(past == 1 ? x.y : past == 2 ? x.z : past == 3 ? x.w : 0.f, past == 1 ? x.z : past == 2 ? x.w : 0.f,
                     past == 1 ? x.w : 0.f, 0.f);
}

// The code of x: fl(x * lambda) rounded to the nearest even integer or towards zero and clamped to [-qmax, qmax], plus 1.5 * 2^23:
// the code in two's complement is the low byte, and code_value the code as a float (the addition rounds to the nearest
// even integer, exactly for what is one already)
constexpr float kCodeBias = 12582912.f;
static __device__ __forceinline__ float biased_code(float x, float lam, float qmax, bool trunc) {
  float y = x * lam;
  if (trunc) y = truncf(y);
  return __builtin_amdgcn_fmed3f(y, -qmax, qmax) + kCodeBias;   // (0 * inf becomes -qmax, as with fminf(fmaxf()))
}
static __device__ __forceinline__ float code_value(float z) { return z - kCodeBias; }
// the low bytes of the first n of four, zeros for the others
static __device__ __forceinline__ unsigned pack_codes(float z0, float z1, float z2, float z3, int n) {
  unsigned p = __builtin_amdgcn_perm(__float_as_uint(z1), __float_as_uint(z0), 0x0c0c0400u);
  p = __builtin_amdgcn_perm(__float_as_uint(z2), p, 0x0c040100u);
  p = __builtin_amdgcn_perm(__float_as_uint(z3), p, 0x04020100u);
  return n >= 4 ? p : p & ((1u << (8 * (n > 0 ? n : 0))) - 1u);
}

static __device__ __forceinline__ void store_part(float* p, const float (&v)[4], int n) {
  if (n >= 4) {
    *reinterpret_cast<f4u*>(p) = f4u{v[0], v[1], v[2], v[3]};
  } else {
    for (int c = 0; c < n; ++c) p[c] = v[c];
  }
}

}  // namespace srq
#endif  // SRQ_STREAM_H_
