// k-major copies of residual codes (element-major: row k holds the codes of all vectors), which the vector-ALU executions of the
// corrections gather from, out of the K-contiguous ones: 2 bytes moved per element, where a pass of fused.hip that writes
// them from the FP32 operand moves 5.
//
// A thread transposes 16 x 16 bytes in registers.  A wave has 8 x 8 of these, so that its loads are 128 contiguous bytes of eight
// vectors and its stores 128 contiguous bytes of eight k.  Nothing is shared; bound by the 2 bytes per element.
#include <cstring>
#include "stream.h"

namespace srq {
namespace {

typedef unsigned u4a __attribute__((ext_vector_type(4)));

// four words of four bytes each, transposed
__device__ __forceinline__ void transpose4(unsigned& a, unsigned& b, unsigned& c, unsigned& d) {
  const unsigned ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const unsigned cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  a = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
  b = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
  c = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
  d = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
}

// a workgroup: 128 elements of 512 vectors
__global__ __launch_bounds__(256) void codes_em_kernel(CodesEm a, CodesEm b, int64_t veclen, int64_t ld, int groups_a, int pieces) {
  const bool first = (int)(blockIdx.x / (unsigned)pieces) < groups_a;
  const CodesEm& o = first ? a : b;
  if (!run_if_ok(o.run)) return;
  const int group = (int)(blockIdx.x / (unsigned)pieces) - (first ? 0 : groups_a), piece = blockIdx.x % (unsigned)pieces;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e0 = (int64_t)piece * 128 + 16 * (lane & 7), v0 = (int64_t)group * 512 + w * 128 + 16 * (lane >> 3);
  if (e0 >= veclen || v0 >= o.nvec) return;
  unsigned x[16][4];                                   // [vector][four elements]
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t v = v0 + i < o.nvec ? v0 + i : o.nvec - 1;
    const u4a t = *reinterpret_cast<const u4a*>(o.R + v * ld + e0);
    x[i][0] = t.x; x[i][1] = t.y; x[i][2] = t.z; x[i][3] = t.w;
  }
  // afterwards word x[4 j + r][c] has element 4 c + r of vectors 4 j .. 4 j + 3
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) transpose4(x[4 * j][c], x[4 * j + 1][c], x[4 * j + 2][c], x[4 * j + 3][c]);
  const int here = (int)(o.nvec - v0 < 16 ? o.nvec - v0 : 16);
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t e = e0 + 4 * c + r;
      if (e >= veclen) continue;
      int8_t* dst = o.Rem + e * o.nvec + v0;
      if (here == 16) {
        const u4u t = {x[r][c], x[4 + r][c], x[8 + r][c], x[12 + r][c]};
        __builtin_nontemporal_store(t, reinterpret_cast<u4u*>(dst));
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = here - 4 * j;
          const unsigned four = x[4 * j + r][c];
          if (n >= 4) {
            *reinterpret_cast<u1u*>(dst + 4 * j) = four;
          } else {
#pragma unroll
            for (int i = 0; i < 3; ++i)
              if (i < n) dst[4 * j + i] = (int8_t)(four >> (8 * i));
          }
        }
      }
    }
}

}  // namespace

hipError_t launch_codes_em(const CodesEm& a, const CodesEm& b, int64_t veclen, int64_t ld, hipStream_t st) {
  const int64_t ga = (a.nvec + 511) / 512, gb = (b.nvec + 511) / 512, pieces = (veclen + 127) / 128;
  if (ga + gb == 0 || pieces == 0) return hipSuccess;
  hipLaunchKernelGGL(codes_em_kernel, dim3((unsigned)((ga + gb) * pieces)), dim3(256), 0, st, a, b, veclen, ld, (int)ga, (int)pieces);
  return hipGetLastError();
}

}  // namespace srq
