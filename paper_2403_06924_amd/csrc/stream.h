// Device functions shared by the streaming kernels over FP32 operands (fused.hip, strips.hip).
#ifndef SRQ_STREAM_H_
#define SRQ_STREAM_H_
#include "srq_internal.h"

namespace srq {

static __device__ __forceinline__ int quant_code(float x, float lam, float qmax, int trunc) {
  float y = x * lam;
  float r = trunc ? truncf(y) : rintf(y);
  r = fminf(fmaxf(r, -qmax), qmax);
  return (int)r;
}

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

static __device__ __forceinline__ void store_part(float* p, const float (&v)[4], int n) {
  if (n >= 4) {
    *reinterpret_cast<f4u*>(p) = f4u{v[0], v[1], v[2], v[3]};
  } else {
    for (int c = 0; c < n; ++c) p[c] = v[c];
  }
}

static __device__ __forceinline__ unsigned pack4(int a, int b, int c, int d) {
  return (unsigned)(a & 0xff) | ((unsigned)(b & 0xff) << 8) | ((unsigned)(c & 0xff) << 16) |
         ((unsigned)(d & 0xff) << 24);
}

}  // namespace srq
#endif  // SRQ_STREAM_H_
