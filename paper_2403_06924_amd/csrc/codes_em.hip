// k-major copies of residual codes (element-major: row k holds the codes of all vectors), which the vector-ALU executions of the
// corrections gather from, out of the K-contiguous ones: 2 bytes moved per element, where a pass of fused.hip that writes
// them from the FP32 operand moves 5.
//
// Behind them the launch that decides, compacts and copies for large calls.
//
// A thread transposes 16 x 16 bytes in registers.  A wave has 8 x 8 of these, so that its loads are 128 contiguous bytes of eight
// vectors and its stores 128 contiguous bytes of eight k.  Nothing is shared; bound by the 2 bytes per element.
#include <cstring>
#include "compact.h"
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

// 128 elements of 512 vectors
__device__ __forceinline__ void copy_block(const CodesEm& o, int group, int piece, int64_t veclen, int64_t ld) {
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

__global__ __launch_bounds__(256) void codes_em_kernel(CodesEm a, CodesEm b, int64_t veclen, int64_t ld, int groups_a, int pieces) {
  const bool first = (int)(blockIdx.x / (unsigned)pieces) < groups_a;
  const CodesEm& o = first ? a : b;
  if (!run_if_ok(o.run)) return;
  copy_block(o, (int)(blockIdx.x / (unsigned)pieces) - (first ? 0 : groups_a), blockIdx.x % (unsigned)pieces, veclen, ld);
}

// ---- Large calls whose executions are decided on the device: the decision, the compaction of both operands and the copies
// that it asks for, in one launch.  The selection has added up the counts of every 256 vectors; each workgroup takes what
// lies before its vectors and the totals, from which it knows the decision, out of these sums and at most 256 counts.
// Measured, us, a scan, a launch for each operand and the copies' / this: 8192 x 8192 each, 5 % kept 77 / 67, 0.1 % 100 / 80 (both
// operands copied), 4096 x 4096 and 4096 x 14336 55 / 34.  Calls: 8192^3 0.1 % 977 / 957, 4096 x 14336 x 4096 809 / 799, 16384^3 20 %
// 10200 / 10120, 5000 x 4000 x 3000 329 / 305, 10000 x 3000 x 2500 371 / 345.
__device__ __forceinline__ int wave_sum(int x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// thread's part of the first n sums
__device__ __forceinline__ int part_of(const int32_t* sums, int n) {
  int x = 0;
  for (int i = threadIdx.x; i < n; i += 256) x += sums[i * kSumStride];
  return x;
}

template <int NV>
__global__ __launch_bounds__(256, NV <= 8 ? 5 : 3) void compact_decide_kernel(CompactDecide g, int K, int Kc) {
  __shared__ int64_t before[4];
  __shared__ int count[4], total[2][4];
  __shared__ __attribute__((aligned(16))) uint8_t gather[4 * kGatherWave];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, id = blockIdx.x;
  const int compact = g.groups_a + g.groups_b;
  const int sums_a = (g.a.nvec + 255) / 256, sums_b = (g.b.nvec + 255) / 256;
  // (totals over both operands, or one of them: int, since either is below 2^31)
  auto totals = [&](bool of_a, bool of_b) __attribute__((always_inline)) {
    const int na = wave_sum(of_a ? part_of(g.sums, sums_a) : 0), nb = wave_sum(of_b ? part_of(g.sums + sums_a * kSumStride, sums_b) : 0);
    if (lane == 0) { total[0][w] = na; total[1][w] = nb; }
    __syncthreads();
  };
  auto kept = [&](int term) __attribute__((always_inline)) -> int64_t { return (int64_t)total[term][0] + total[term][1] + total[term][2] + total[term][3]; };
  if (id < compact) {
    const bool second = id >= g.groups_a;
    const StripCompact& s = second ? g.b : g.a;
    const int group = second ? id - g.groups_a : id, v0 = 4 * group;
    CompactFour<NV> f;
    f.load(s, group, K, Kc);
    int sum = part_of(second ? g.sums + sums_a * kSumStride : g.sums, v0 >> 8);
    const int i = (v0 & ~255) + (int)threadIdx.x;
    if (i < v0) sum += s.counts[i];
    sum = wave_sum(sum);
    if (lane == 0) before[w] = sum;
    totals(!second || id == 0, second || id == 0);
    f.store(s, kept(second) >= (second ? g.dec.min_mfma_b : g.dec.min_mfma_a) ? s.dense : nullptr, K, Kc, before, count, gather, g.around);
    if (id == 0 && threadIdx.x == 0) {
      const int64_t na = kept(0), nb = kept(1);
      const int pa = g.a.nvec ? (na >= g.dec.min_mfma_a ? 2 : 1) : 0, pb = g.b.nvec ? (nb >= g.dec.min_mfma_b ? 2 : 1) : 0;
      g.dec.paths[0] = pa;
      g.dec.paths[1] = pb;
      if (g.dec.seen && pa) g.dec.seen[0] = pa;
      if (g.dec.seen && pb) g.dec.seen[1] = pb;
      if (g.dec.stats) {
        g.dec.stats->nnz_a = na;
        g.dec.stats->nnz_b = nb;
        g.dec.stats->path_a = pa;
        g.dec.stats->path_b = pb;
        g.dec.stats->overflow = (na > g.dec.cap_a ? 1 : 0) | (nb > g.dec.cap_b ? 2 : 0);
        g.dec.stats->reserved = 0;
      }
    }
    return;
  }
  // the residual codes of A feed term 2, whose execution the entries of B decide; those of B term 1
  const int pieces = (K + 127) / 128, group = (id - compact) / pieces, piece = (id - compact) % pieces;
  const int em_a = (int)((g.em_a.nvec + 511) / 512);
  const bool of_a = group < em_a;
  if (of_a ? !g.always_a : !g.always_b) {
    totals(!of_a, of_a);
    if (of_a ? kept(1) >= g.dec.min_mfma_b : kept(0) >= g.dec.min_mfma_a) return;
  }
  copy_block(of_a ? g.em_a : g.em_b, of_a ? group : group - em_a, piece, K, Kc);
}

}  // namespace

hipError_t launch_codes_em(const CodesEm& a, const CodesEm& b, int64_t veclen, int64_t ld, hipStream_t st) {
  const int64_t ga = (a.nvec + 511) / 512, gb = (b.nvec + 511) / 512, pieces = (veclen + 127) / 128;
  if (ga + gb == 0 || pieces == 0) return hipSuccess;
  hipLaunchKernelGGL(codes_em_kernel, dim3((unsigned)((ga + gb) * pieces)), dim3(256), 0, st, a, b, veclen, ld, (int)ga, (int)pieces);
  return hipGetLastError();
}

hipError_t launch_compact_decide(const CompactDecide& with, int64_t K, int64_t Kc, hipStream_t st) {
  CompactDecide g = with;
  g.groups_a = (g.a.nvec + 3) / 4;
  g.groups_b = (g.b.nvec + 3) / 4;
  // zero-filled codes past what the last-level cache keeps until they are read, calls, us, through the caches / around them:
  // 8192^3 1437 / 1428, 16384^3 10285 / 10281, but 4096 x 14336 x 4096 802 / 806, 5000 x 4000 x 3000 324 / 328
  g.around = ((int64_t)g.a.nvec + g.b.nvec) * K > 100000000;
  const int64_t copies = ((g.em_a.nvec + 511) / 512 + (g.em_b.nvec + 511) / 512) * ((K + 127) / 128);
  const dim3 grid((unsigned)(g.groups_a + g.groups_b + copies));
  if (Kc <= 2048) hipLaunchKernelGGL(compact_decide_kernel<2>, grid, dim3(256), 0, st, g, (int)K, (int)Kc);
  else if (Kc <= 4096) hipLaunchKernelGGL(compact_decide_kernel<4>, grid, dim3(256), 0, st, g, (int)K, (int)Kc);
  else if (Kc <= 8192) hipLaunchKernelGGL(compact_decide_kernel<8>, grid, dim3(256), 0, st, g, (int)K, (int)Kc);
  else hipLaunchKernelGGL(compact_decide_kernel<16>, grid, dim3(256), 0, st, g, (int)K, (int)Kc);
  return hipGetLastError();
}

}  // namespace srq
