// The passes over the operands for a short inner dimension, or few rows and columns (strips_ok), where one
// workgroup can hold whole columns of B: what takes ten launches on the kernels of fused.hip and
// select.hip takes three here.
//
//   quant_pair_kernel    both operands in one launch and one read of each: maxima, scales, codes, residual
//                        scales and residual codes.  A workgroup has either rows of A in registers or a
//                        strip of 4 * CG columns of B over all of K (TH / CG pieces of RPT rows).
//   select_pair_kernel   means of |D_F| from the partial sums, thresholds, keep-masks and counts of both
//                        operands, cut in the same way (no atomics, nothing to clear); beyond K = 1024 for thresholds and
//                        codes that select_codes.hip does not take.
//   quant_cols_kernel, reduce_rows_kernel, reduce_cols_kernel   the staged entry points on one operand
//   compact_pair_kernel  compaction to CSR / CSC and to zero-filled codes of both operands; every workgroup
//                        adds up the counts before its vector itself, so that no scan runs in between (behind the
//                        tiles of the corrections where they are 64 x 64, gemm_tile64.hip).
//
// What bounds them: at these sizes the latency of a launch and of one trip through a workgroup, not
// bandwidth; hence few elements per thread for short K (RPT 4 or 8) and as many workgroups as there are.
// A strip reads 64, 32 or 16 bytes of each row of B; strips that share 128-byte lines are given to the same
// XCD (strip_of), where the line is found in L2 the second time.
// Up to K = 4096 a wave has a row of A to itself: nothing in a row then waits at a barrier, and the workgroups are a quarter to an
// eighth as many.  With a workgroup per row / a wave: 2048^3 quantize 17.6 / 13.3 us, 2048^2 x 2112 30 / 22.
// (the kernel for K beyond 2048 needs 188 registers, its strips 162).
#include "compact.h"
#include "stream.h"

namespace srq {
namespace {

// (kGroup: neighbouring strips handed to one XCD)
template <int kGroup>
__device__ __forceinline__ int strip_of(int b, int strips) {
  if (b >= strips / (8 * kGroup) * (8 * kGroup)) return b;
  const int q = b >> 3, x = b & 7;                   // workgroup b runs on XCD b % 8
  return ((q / kGroup) * 8 + x) * kGroup + q % kGroup;
}

typedef unsigned u2u __attribute__((ext_vector_type(2), aligned(1)));

__device__ __forceinline__ float4 abs4(float4 x) { return make_float4(fabsf(x.x), fabsf(x.y), fabsf(x.z), fabsf(x.w)); }
__device__ __forceinline__ float max4(float4 x) { return fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)); }

// TH threads, sm: TH / 64 words
template <int TH>
__device__ __forceinline__ float block_max(float m, float* sm) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  __syncthreads();                                   // sm may still be read from a previous use
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
  __syncthreads();
  m = sm[0];
#pragma unroll
  for (int i = 1; i < TH / 64; ++i) m = fmaxf(m, sm[i]);
  return m;
}

// The NV4 pieces of a row that thread t of RT has (every RT-th four values), zeros past K
template <int RT, int NV4>
__device__ __forceinline__ void load_row(float4 (&x)[NV4], int (&n)[NV4], const float* src, int K, int t) {
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int e = 4 * (t + i * RT);
    n[i] = K - e >= 4 ? 4 : K - e > 0 ? K - e : 0;
  }
  if (K < 4) {
#pragma unroll
    for (int i = 0; i < NV4; ++i) x[i] = load_part(src + 4 * (t + i * RT), n[i]);
    return;
  }
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const f4u y = load_inside(src, 4 * (t + i * RT), K);
    x[i] = make_float4(y.x, y.y, y.z, y.w);
  }
  if (K < 4 * RT * NV4) {                            // (somebody reaches past K)
#pragma unroll
    for (int i = 0; i < NV4; ++i) x[i] = shifted(f4u{x[i].x, x[i].y, x[i].z, x[i].w}, 4 * (t + i * RT), K);
  }
}
// A thread's patch of a strip: rows row0 .. row0 + RPT - 1 of four columns from col0 on, zeros outside.  (Put right in place,
// under one branch: with both forms behind an if and else the selection takes 147 registers for 116, one workgroup on a
// compute unit for two; 2999 x 4097 x 3001 245 us / 239.)
template <int TH, int CG, int RPT>
__device__ __forceinline__ void load_patch(float4 (&v)[RPT], const float* X, int64_t ldx, int strip, int row0, int64_t col0, int64_t cols,
                                           int K) {
  if (cols < 4) {
    const int n = (int)(cols - col0);
#pragma unroll
    for (int i = 0; i < RPT; ++i) v[i] = load_part(X + (int64_t)(row0 + i) * ldx + col0, row0 + i < K ? n : 0);
    return;
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const f4u t = load_inside(X + (int64_t)(row0 + i < K ? row0 + i : K - 1) * ldx, (int)col0, (int)cols);
    v[i] = make_float4(t.x, t.y, t.z, t.w);
  }
  if (K < TH / CG * RPT || (int64_t)(strip + 1) * 4 * CG > cols) {   // (part of the strip does not exist)
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      v[i] = shifted(f4u{v[i].x, v[i].y, v[i].z, v[i].w}, (int)col0, (int)cols);
      if (row0 + i >= K) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
}

// maximum over the RT threads of a row: a wave or the workgroup
template <int RT>
__device__ __forceinline__ float row_max(float m, float* sm) {
  if constexpr (RT > 64) return block_max<RT>(m, sm);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  return m;
}

// ---- quantization ----------------------------------------------------------------------------------
// One row by RT threads, a wave (no barriers) or the whole workgroup.  Codes go out up to the padded length (zeros past K); places past K stay out of the maxima of
// the residual (0 * lam is not 0 where lam overflowed).
template <int RT, int NV4>
__device__ __forceinline__ void quant_row(const StripOperand& s, int64_t row, int K, int Kc, float qmax, int trunc, float* sm) {
  const int t = threadIdx.x & (RT - 1);
  float4 x[NV4];
  int n[NV4];
  float m = 0.f;
  load_row<RT, NV4>(x, n, s.X + row * s.ldx, K, t);
#pragma unroll
  for (int i = 0; i < NV4; ++i) m = fmaxf(m, max4(abs4(x[i])));
  if (s.nonzero) {                                   // (as a float: no row is longer than 8192)
    int some = 0;
#pragma unroll
    for (int i = 0; i < NV4; ++i)
      some += (fabsf(x[i].x) > 0.f) + (fabsf(x[i].y) > 0.f) + (fabsf(x[i].z) > 0.f) + (fabsf(x[i].w) > 0.f);
    for (int off = 32; off > 0; off >>= 1) some += __shfl_xor(some, off, 64);
    if constexpr (RT > 64) {
      if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = (float)some;
      __syncthreads();
      float all = 0.f;
      for (int i = 0; i < RT / 64; ++i) all += sm[i];
      some = (int)all;
    }
    if (t == 0) s.nonzero[row] = some;
  }
  const float amax = row_max<RT>(m, sm);
  float lam = 0.f, sc = 0.f;
  if (amax > 0.f) { lam = qmax / amax; sc = amax / qmax; }
  float rm = 0.f;
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int e = 4 * (t + i * RT);
    float v[4] = {x[i].x, x[i].y, x[i].z, x[i].w}, z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      z[j] = biased_code(v[j], lam, qmax, trunc);
      v[j] = j < n[i] ? v[j] - code_value(z[j]) * sc : 0.f;
      rm = fmaxf(rm, fabsf(v[j]));
    }
    if (e < Kc) *reinterpret_cast<unsigned*>(s.Q + row * Kc + e) = pack_codes(z[0], z[1], z[2], z[3], n[i]);
    x[i] = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (t == 0) { s.scale[row] = sc; s.lambda[row] = lam; }
  if (!s.Rq) return;
  const float ramax = row_max<RT>(rm, sm);
  float rlam = 0.f, rs = 0.f;
  if (ramax > 0.f) { rlam = qmax / ramax; rs = ramax / qmax; }
  if (t == 0) { s.rscale[row] = rs; s.rlambda[row] = rlam; }
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int e = 4 * (t + i * RT);
    const float v[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
    float z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = biased_code(v[j], rlam, qmax, trunc);
    if (e < Kc) *reinterpret_cast<unsigned*>(s.Rq + row * Kc + e) = pack_codes(z[0], z[1], z[2], z[3], n[i]);
  }
  for (int e = K + t; e < Kc; e += RT) s.D[row * Kc + e] = 0;
}

// maxima of the CG * 4 columns of a strip from every thread's own four; red: [TH / 64][4 * CG]
template <int TH, int CG>
__device__ __forceinline__ void strip_max(float (&m)[4], float* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cg = threadIdx.x & (CG - 1);
#pragma unroll
  for (int off = CG; off < 64; off <<= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], __shfl_xor(m[c], off, 64));
  if (lane < CG)
#pragma unroll
    for (int c = 0; c < 4; ++c) red[w * 4 * CG + cg * 4 + c] = m[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c)
    for (int i = 0; i < TH / 64; ++i) m[c] = fmaxf(m[c], red[(i * CG + cg) * 4 + c]);
}

// RPT codes of each of the patch's columns: Q[col * ld + row0 ..], places from `lim` on left alone
template <int RPT>
__device__ __forceinline__ void store_codes(int8_t* Q, int64_t ld, int lim, int64_t col0, int ncol, int row0,
                                            const unsigned (&pk)[4][RPT / 4]) {
  if (row0 >= lim) return;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (c >= ncol) break;
    int8_t* dst = Q + (col0 + c) * ld + row0;
    if (row0 + RPT <= lim) {
      if constexpr (RPT == 16) *reinterpret_cast<u4u*>(dst) = u4u{pk[c][0], pk[c][1], pk[c][2], pk[c][3]};
      else if constexpr (RPT == 8) *reinterpret_cast<u2u*>(dst) = u2u{pk[c][0], pk[c][1]};
      else *reinterpret_cast<u1u*>(dst) = pk[c][0];
    } else {
#pragma unroll
      for (int i = 0; i < RPT; ++i)
        if (row0 + i < lim) dst[i] = (int8_t)(pk[c][i >> 2] >> (8 * (i & 3)));
    }
  }
}

// codes of a patch, zeros from row K on; RESID: the patch becomes its residual, rm its columns' maxima
template <int RPT, bool RESID>
__device__ __forceinline__ void patch_codes(float4 (&v)[RPT], const float (&lam)[4], const float (&sc)[4], float qmax, bool trunc, int left,
                                            unsigned (&pk)[4][RPT / 4], float (&rm)[4]) {
#pragma unroll
  for (int i = 0; i < RPT; i += 4) {
    float z[4][4];                                   // [row][column]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x[4] = {v[i + r].x, v[i + r].y, v[i + r].z, v[i + r].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        z[r][c] = biased_code(x[c], lam[c], qmax, trunc);
        if (RESID) {
          x[c] = i + r < left ? x[c] - code_value(z[r][c]) * sc[c] : 0.f;   // (0 * lam is not 0 where lam overflowed)
          rm[c] = fmaxf(rm[c], fabsf(x[c]));
        }
      }
      if (RESID) v[i + r] = make_float4(x[0], x[1], x[2], x[3]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) pk[c][i / 4] = pack_codes(z[0][c], z[1][c], z[2][c], z[3][c], left - i);
    __builtin_amdgcn_sched_barrier(0);               // (all rows at once would take 60 more registers)
  }
}

template <int TH, int CG, int RPT, bool COUNT>   // COUNT: entries that are not zero, if wanted
__device__ __forceinline__ void quant_strip(const StripOperand& s, int strip, int64_t cols, int K, int Kc, int64_t ldq, float qmax,
                                            int trunc, float* red) {
  const int cg = threadIdx.x & (CG - 1), rb = threadIdx.x / CG, row0 = rb * RPT;
  const int64_t col0 = ((int64_t)strip * CG + cg) * 4;
  const int ncol = col0 + 4 <= cols ? 4 : col0 < cols ? (int)(cols - col0) : 0;
  float4 v[RPT];
  float m[4] = {0.f, 0.f, 0.f, 0.f};
  load_patch<TH, CG, RPT>(v, s.X, s.ldx, strip, row0, col0, cols, K);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const float4 a = abs4(v[i]);
    m[0] = fmaxf(m[0], a.x); m[1] = fmaxf(m[1], a.y); m[2] = fmaxf(m[2], a.z); m[3] = fmaxf(m[3], a.w);
  }
  __shared__ int some[COUNT ? 4 * CG : 1];
  if (COUNT && s.nonzero) {                          // (through LDS at once: four registers more cost 1024 x 1024 2 % of a call)
    if ((int)threadIdx.x < 4 * CG) some[threadIdx.x] = 0;
    __syncthreads();
    int n[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      n[0] += fabsf(v[i].x) > 0.f; n[1] += fabsf(v[i].y) > 0.f;
      n[2] += fabsf(v[i].z) > 0.f; n[3] += fabsf(v[i].w) > 0.f;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) atomicAdd(&some[cg * 4 + c], n[c]);
  }
  strip_max<TH, CG>(m, red);
  float lam[4], sc[4], rm[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lam[c] = m[c] > 0.f ? qmax / m[c] : 0.f;
    sc[c] = m[c] > 0.f ? m[c] / qmax : 0.f;
  }
  if (rb == 0) { store_part(s.scale + col0, sc, ncol); store_part(s.lambda + col0, lam, ncol); }
  unsigned pk[4][RPT / 4];
  patch_codes<RPT, true>(v, lam, sc, qmax, trunc, K - row0, pk, rm);
  store_codes<RPT>(s.Q, ldq, Kc, col0, ncol, row0, pk);
  if (!s.Rq) return;
  strip_max<TH, CG>(rm, red + TH / 16 * CG);
  if (COUNT && s.nonzero && rb == 0)
    for (int c = 0; c < ncol; ++c) s.nonzero[col0 + c] = some[cg * 4 + c];
  float rlam[4], rs[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    rlam[c] = rm[c] > 0.f ? qmax / rm[c] : 0.f;
    rs[c] = rm[c] > 0.f ? rm[c] / qmax : 0.f;
  }
  if (rb == 0) { store_part(s.rscale + col0, rs, ncol); store_part(s.rlambda + col0, rlam, ncol); }
  patch_codes<RPT, false>(v, rlam, rs, qmax, trunc, K - row0, pk, rm);
  store_codes<RPT>(s.Rq, ldq, Kc, col0, ncol, row0, pk);
  for (int i = threadIdx.x; i < 4 * CG * (Kc - K); i += TH) {
    const int64_t col = (int64_t)strip * 4 * CG + i / (Kc - K);
    if (col < cols) s.D[col * Kc + K + i % (Kc - K)] = 0;
  }
}

template <int TH, int RT, int NV4, int CG, int RPT>
__global__ __launch_bounds__(TH) void quant_pair_kernel(StripOperand a, StripOperand b, int64_t M, int64_t N, int K, int Kc, int strips,
                                                         float qmax, int trunc) {
  __shared__ float sm[TH / 8 * CG];
  const int64_t row = ((int64_t)blockIdx.x - strips) * (TH / RT) + (RT == 64 ? threadIdx.x >> 6 : 0);
  if ((int)blockIdx.x < strips) quant_strip<TH, CG, RPT, true>(b, strip_of<8 / CG>(blockIdx.x, strips), N, K, Kc, Kc, qmax, trunc, sm);
  else if (row < M) quant_row<RT, NV4>(a, row, K, Kc, qmax, trunc, sm);
}

// columns alone, into a caller's matrix of any leading dimension
template <int TH, int RT, int NV4, int CG, int RPT>
__global__ __launch_bounds__(TH) void quant_cols_kernel(StripOperand s, int64_t N, int K, int64_t ldq, int strips, float qmax,
                                                        int trunc) {
  __shared__ float sm[TH / 8 * CG];
  quant_strip<TH, CG, RPT, false>(s, strip_of<8 / CG>(blockIdx.x, strips), N, K, K, ldq, qmax, trunc, sm);
}

// ---- selection -------------------------------------------------------------------------------------
__device__ __forceinline__ void mean_of(const StripSelect& s, int64_t v, double sum, bool writer, float& t) {
  const float mean = (float)(sum / s.count);
  t = s.theta * mean;
  if (writer) {
    s.mean[v] = mean;
    s.thresh[v] = t;
    if (!s.mask && s.counts && t != t) s.counts[v] = 0;
  }
}

// eight neighbouring lanes assemble one 32-bit piece of a row's mask
__device__ __forceinline__ void store_nibble(uint64_t* mrow, int words, int c4, unsigned nib) {
  const unsigned b8 = nib | (__shfl_down(nib, 1, 64) << 4);
  const unsigned b16 = b8 | (__shfl_down(b8, 2, 64) << 8);
  const unsigned b32 = b16 | (__shfl_down(b16, 4, 64) << 16);
  if (!(c4 & 7) && (c4 >> 3) < 2 * words) reinterpret_cast<uint32_t*>(mrow)[c4 >> 3] = b32;
}

// The partial sums of a vector, K > 1024: every 64th by a lane, the lanes as a tree, in this order wherever such a call forms
// its means (select_codes.hip), each wave that wants the sum by itself.  (Up to 1024: see select_strip; a wave has a row.)
__device__ __forceinline__ double sum_of(const StripSelect& s, int64_t v, int64_t nvec) {
  double sum = 0.0;
  for (int64_t p = threadIdx.x & 63; p < s.nparts; p += 64) sum += s.part[p * nvec + v];
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  return sum;
}

template <int RT, int NV4>
__device__ __forceinline__ void select_row(const StripSelect& s, int64_t row, int64_t rows, int K, int* ism) {
  const int tid = threadIdx.x & (RT - 1), lane = tid & 63, w = tid >> 6;
  const int words = (K + 63) / 64;
  float4 x[NV4];
  int n[NV4];
  if (s.mask) load_row<RT, NV4>(x, n, s.X + row * s.ldx, K, tid);   // (on their way while the threshold is formed)
  constexpr bool kDense = RT == 64 && NV4 <= 4;        // K <= 1024
  unsigned code[kDense ? NV4 : 1];
  if (kDense && s.D) {
#pragma unroll
    for (int i = 0; i < NV4; ++i) {
      const int e = 4 * (tid + i * RT);
      code[kDense ? i : 0] = *reinterpret_cast<const unsigned*>(s.Q + row * s.ldq + (e < s.ldq ? e : 0));
    }
  }
  const double sum = sum_of(s, row, rows);
  float t;
  mean_of(s, row, sum, tid == 0, t);
  if (!s.mask) return;
  int total = 0;
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int c4 = tid + i * RT;
    unsigned nib = (fabsf(x[i].x) > t ? 1u : 0u) | (fabsf(x[i].y) > t ? 2u : 0u) | (fabsf(x[i].z) > t ? 4u : 0u) |
                   (fabsf(x[i].w) > t ? 8u : 0u);
    nib &= (1u << n[i]) - 1u;
    total += __popc(nib);
    store_nibble(s.mask + row * words, words, c4, nib);
    if (kDense && s.D && 4 * c4 < s.ldq) *reinterpret_cast<unsigned*>(s.D + row * s.ldq + 4 * c4) = code[kDense ? i : 0] & bytes_of(nib);
  }
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
  if constexpr (RT > 64) {
    if (lane == 0) ism[w] = total;
    __syncthreads();
    total = ism[0];
#pragma unroll
    for (int i = 1; i < RT / 64; ++i) total += ism[i];
  }
  if (tid == 0) s.counts[row] = total;
}

// keep-bits of a patch (bit i of bits[c]: row row0 + i of column c) into the mask, and the counts of the strip's columns
template <int TH, int CG, int RPT>
__device__ __forceinline__ void store_bits(uint64_t* mask, int32_t* counts, int strip, int64_t cols, int K, int64_t col0, int ncol,
                                           const unsigned (&bits)[4], int* ism) {
  constexpr int BC = 4 * CG;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, cg = tid & (CG - 1), rb = tid / CG, row0 = rb * RPT;
  const int words = (K + 63) / 64;
  int cnt[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cnt[c] = c < ncol ? __popc(bits[c]) : 0;
    unsigned piece = bits[c];
    if constexpr (RPT == 4) piece |= __shfl_down(piece, CG, 64) << 4;     // two threads' rows make one byte
    if (c < ncol && row0 < words * 64) {
      uint8_t* dst = reinterpret_cast<uint8_t*>(mask + (col0 + c) * words) + (row0 >> 3);
      if constexpr (RPT == 16) *reinterpret_cast<uint16_t*>(dst) = (uint16_t)piece;
      else if constexpr (RPT == 8) *dst = (uint8_t)piece;
      else if (!(rb & 1)) *dst = (uint8_t)piece;
    }
  }
#pragma unroll
  for (int off = CG; off < 64; off <<= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) cnt[c] += __shfl_xor(cnt[c], off, 64);
  if (lane < CG)
#pragma unroll
    for (int c = 0; c < 4; ++c) ism[w * BC + cg * 4 + c] = cnt[c];
  __syncthreads();
  if (tid < BC && (int64_t)strip * BC + tid < cols) {
    int total = ism[tid];
#pragma unroll
    for (int i = 1; i < TH / 64; ++i) total += ism[i * BC + tid];
    counts[(int64_t)strip * BC + tid] = total;
  }
}

template <int TH, int CG, int RPT>
__device__ __forceinline__ void select_strip(const StripSelect& s, int strip, int64_t cols, int K, double* dsm, int* ism) {
  constexpr int BC = 4 * CG;
  constexpr bool kWaveSums = TH / CG * RPT > 1024;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, cg = tid & (CG - 1), rb = tid / CG, row0 = rb * RPT;
  const int words = (K + 63) / 64;
  const int64_t col0 = ((int64_t)strip * CG + cg) * 4;
  const int ncol = col0 + 4 <= cols ? 4 : col0 < cols ? (int)(cols - col0) : 0;
  float4 v[RPT];
  if (s.mask) load_patch<TH, CG, RPT>(v, s.X, s.ldx, strip, row0, col0, cols, K);
  constexpr int kDense = !kWaveSums && RPT <= 8 ? RPT / 4 : 0;   // words of codes per column, K <= 1024
  unsigned code[4][kDense ? kDense : 1];
  if (kDense && s.D) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const unsigned* src = reinterpret_cast<const unsigned*>(s.Q + (col0 + c < cols ? col0 + c : cols - 1) * s.ldq + (row0 < s.ldq ? row0 : 0));
#pragma unroll
      for (int i = 0; i < kDense; ++i) code[c][i] = src[i];
    }
  }
  if constexpr (kWaveSums) {
    for (int c = w; c < BC; c += TH / 64) {
      const int64_t pc = (int64_t)strip * BC + c;
      const double sum = pc < cols ? sum_of(s, pc, cols) : 0.0;
      if (lane == 0) dsm[c] = sum;
    }
  } else {
    // partial sums: BC neighbouring columns by BC neighbouring threads
    const int64_t pc = (int64_t)strip * BC + (tid & (BC - 1));
    double sum = 0.0;
    if (pc < cols)
      for (int64_t p = tid / BC; p < s.nparts; p += TH / BC) sum += s.part[p * cols + pc];
#pragma unroll
    for (int off = BC; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
    if (lane < BC) dsm[w * BC + lane] = sum;
  }
  __syncthreads();
  float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double all = dsm[cg * 4 + c];
    if constexpr (!kWaveSums) {
#pragma unroll
      for (int i = 1; i < TH / 64; ++i) all += dsm[i * BC + cg * 4 + c];
    }
    if (c < ncol) mean_of(s, col0 + c, all, rb == 0, t[c]);
  }
  if (!s.mask) return;
  unsigned bits[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const float4 a = abs4(v[i]);
    const bool ok = row0 + i < K;
    bits[0] |= ok && a.x > t[0] ? 1u << i : 0u;
    bits[1] |= ok && a.y > t[1] ? 1u << i : 0u;
    bits[2] |= ok && a.z > t[2] ? 1u << i : 0u;
    bits[3] |= ok && a.w > t[3] ? 1u << i : 0u;
  }
  if (kDense && s.D && row0 < s.ldq) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= ncol) break;
      unsigned* dst = reinterpret_cast<unsigned*>(s.D + (col0 + c) * s.ldq + row0);
#pragma unroll
      for (int i = 0; i < kDense; ++i) dst[i] = code[c][i] & bytes_of(bits[c] >> (4 * i) & 15u);
    }
  }
  store_bits<TH, CG, RPT>(s.mask, s.counts, strip, cols, K, col0, ncol, bits, ism);
}

template <int TH, int RT, int NV4, int CG, int RPT>
__global__ __launch_bounds__(TH) void select_pair_kernel(StripSelect a, StripSelect b, int64_t M, int64_t N, int K, int strips) {
  __shared__ double dsm[TH / 16 * CG];
  __shared__ int ism[TH / 16 * CG];
  const int64_t row = ((int64_t)blockIdx.x - strips) * (TH / RT) + (RT == 64 ? threadIdx.x >> 6 : 0);
  if ((int)blockIdx.x < strips) select_strip<TH, CG, RPT>(b, strip_of<8 / CG>(blockIdx.x, strips), N, K, dsm, ism);
  else if (row < M) select_row<RT, NV4>(a, row, M, K, ism);
}

// ---- reduction of one operand (scales and thresholds given): codes, residual codes, keep-mask and counts in
// one read.  Codes go to rows of Kc bytes with zeros past K, residual codes to the caller's matrix.
template <int TH, int NV4>
__global__ __launch_bounds__(TH) void reduce_rows_kernel(StripReduce s, int K, int Kc, float qmax, int trunc) {
  __shared__ float sm[TH / 64];
  __shared__ int ism[TH / 64];
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, words = (K + 63) / 64;
  const float* src = s.X + row * s.ldx;
  const float lam = s.lambda[row], sc = s.scale[row], t = s.thresh[row];
  float4 x[NV4];
  int n[NV4], total = 0;
  float rm = 0.f;
  load_row<TH, NV4>(x, n, src, K, tid);
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int e = 4 * (tid + i * TH);
    float v[4] = {x[i].x, x[i].y, x[i].z, x[i].w}, z[4];
    unsigned nib = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      nib |= j < n[i] && fabsf(v[j]) > t ? 1u << j : 0u;
      z[j] = biased_code(v[j], lam, qmax, trunc);
      v[j] = j < n[i] ? v[j] - code_value(z[j]) * sc : 0.f;
      rm = fmaxf(rm, fabsf(v[j]));
    }
    total += __popc(nib);
    store_nibble(s.mask + row * words, words, e >> 2, nib);
    if (e < Kc) *reinterpret_cast<unsigned*>(s.Q + row * Kc + e) = pack_codes(z[0], z[1], z[2], z[3], n[i]);
    x[i] = make_float4(v[0], v[1], v[2], v[3]);
  }
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
  if (lane == 0) ism[w] = total;
  const float ramax = block_max<TH>(rm, sm);         // (its barriers publish ism as well)
  float rlam = 0.f, rs = 0.f;
  if (ramax > 0.f) { rlam = qmax / ramax; rs = ramax / qmax; }
  if (tid == 0) {
    total = ism[0];
#pragma unroll
    for (int i = 1; i < TH / 64; ++i) total += ism[i];
    s.counts[row] = total;
    s.rscale[row] = rs;
  }
#pragma unroll
  for (int i = 0; i < NV4; ++i) {
    const int e = 4 * (tid + i * TH);
    const unsigned p = pack_codes(biased_code(x[i].x, rlam, qmax, trunc), biased_code(x[i].y, rlam, qmax, trunc),
                                  biased_code(x[i].z, rlam, qmax, trunc), biased_code(x[i].w, rlam, qmax, trunc), 4);
    int8_t* dst = s.Rq + row * s.ldr + e;
    if (n[i] == 4) {
      *reinterpret_cast<u1u*>(dst) = p;
    } else {
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (j < n[i]) dst[j] = (int8_t)(p >> (8 * j));
    }
  }
}

template <int TH, int RT, int NV4, int CG, int RPT>
__global__ __launch_bounds__(TH) void reduce_cols_kernel(StripReduce s, int64_t cols, int K, int Kc, int strips, float qmax,
                                                         int trunc) {
  __shared__ float red[TH / 16 * CG];
  __shared__ int ism[TH / 16 * CG];
  const int strip = strip_of<8 / CG>(blockIdx.x, strips);
  const int cg = threadIdx.x & (CG - 1), rb = threadIdx.x / CG, row0 = rb * RPT;
  const int64_t col0 = ((int64_t)strip * CG + cg) * 4;
  const int ncol = col0 + 4 <= cols ? 4 : col0 < cols ? (int)(cols - col0) : 0;
  float4 v[RPT];
  load_patch<TH, CG, RPT>(v, s.X, s.ldx, strip, row0, col0, cols, K);
  const float4 l4 = load_part(s.lambda + col0, ncol), s4 = load_part(s.scale + col0, ncol), t4 = load_part(s.thresh + col0, ncol);
  const float lam[4] = {l4.x, l4.y, l4.z, l4.w}, sc[4] = {s4.x, s4.y, s4.z, s4.w}, t[4] = {t4.x, t4.y, t4.z, t4.w};
  float rm[4] = {0.f, 0.f, 0.f, 0.f};
  unsigned bits[4] = {0, 0, 0, 0}, pk[4][RPT / 4];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const float4 a = abs4(v[i]);
    const bool ok = row0 + i < K;
    bits[0] |= ok && a.x > t[0] ? 1u << i : 0u;
    bits[1] |= ok && a.y > t[1] ? 1u << i : 0u;
    bits[2] |= ok && a.z > t[2] ? 1u << i : 0u;
    bits[3] |= ok && a.w > t[3] ? 1u << i : 0u;
  }
  patch_codes<RPT, true>(v, lam, sc, qmax, trunc, K - row0, pk, rm);
  store_codes<RPT>(s.Q, Kc, Kc, col0, ncol, row0, pk);
  store_bits<TH, CG, RPT>(s.mask, s.counts, strip, cols, K, col0, ncol, bits, ism);
  strip_max<TH, CG>(rm, red);
  float rlam[4], rs[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    rlam[c] = rm[c] > 0.f ? qmax / rm[c] : 0.f;
    rs[c] = rm[c] > 0.f ? rm[c] / qmax : 0.f;
  }
  if (rb == 0) store_part(s.rscale + col0, rs, ncol);
  patch_codes<RPT, false>(v, rlam, rs, qmax, trunc, RPT, pk, rm);
  store_codes<RPT>(s.Rq, s.ldr, K, col0, ncol, row0, pk);
}

// ---- compaction ------------------------------------------------------------------------------------
template <int NV>                                      // see compact.h
__global__ __launch_bounds__(256) void compact_pair_kernel(StripCompact a, StripCompact b, int groups_a, int K, int Kc) {
  __shared__ int64_t before[4];
  __shared__ int count[4];
  __shared__ __attribute__((aligned(16))) uint8_t gather[4 * kGatherWave];
  const bool second = (int)blockIdx.x >= groups_a;
  compact_four<NV>(second ? b : a, (int)blockIdx.x - (second ? groups_a : 0), K, Kc, before, count, gather);
}

// a strip of B is 4 * CG columns wide
int strip_cg(int64_t K) { return K <= 512 ? 4 : K <= 4096 ? 2 : 1; }

}  // namespace

// Where the lines lie (calls at 5 % kept, us, streaming kernels / these).  Wider strips of a longer K hold
// more of a compute unit and read narrower pieces of each row, so what launches cost has to be a larger
// share of the call:
//   K <= 1024, any size    512^2 x 256 49 / 26, 8192^2 x 1024 540 / 521
// Against B in one read and the selection from the codes, us, those / these:
//   K <= 1600              10000^2 x 1500 830 / 813, 6000 x 3000 x 1600 248 / 235
//   K <= 2048              4096^2 x 2048 200 / 191, 3000^2 x 2000 154 / 140, 20000 x 200 x 2000 206 / 184; 5000^2 x 2000 298 / 303,
//   and N K <= 8.5e6       8192^2 x 2048 607 / 626
//   K <= 4096              2500^2 x 2300 127 / 122, 3000^2 x 2700 190 / 187, 4500 x 1400 x 4000 174 / 167; 3500^2 x 2500 200 / 201,
//   and N K <= 8.5e6       2000 x 6000 x 3000 226 / 229, 2999 x 4097 x 3001 225 / 230
//   and (M + N) K <= 24e6
//   M + N <= 2048          300^2 x 8000 99 / 92, 300 x 400 x 6000 86 / 79, 900 x 1000 x 8191 123 / 123
bool strips_ok(int64_t M, int64_t N, int64_t K) {
  if (K <= 0 || K > kStripsMaxK || M + N >= (1 << 24)) return false;
  return K <= 1024 || (K <= 1600 && M + N <= 20480) || (K <= 2048 && M + N <= 20480 && N * K <= 8500000) ||
         (K <= 4096 && (M + N) * K <= 24000000 && N * K <= 8500000) || M + N <= 2048;
}
// One operand, srq_quantize and srq_build_sparse_residual with 5 % kept (us, the kernels of cols_once.hip resp. fused.hip / here;
// about 31 us of the small ones is the host): columns 800 x 800 40 / 31, 1000 x 10000 64 / 48, 2000 x 6000 62 / 52, 2000 x 15000 140 /
// 124, 2048 x 25000 218 / 215, 3000 x 1500 42 / 37, 4096 x 2000 43 / 43, 4096 x 5000 74 / 99, 3000 x 9000 125 / 147, 4096 x 10000
// 125 / 167; rows 10000 x 1000 62 / 46, 15000 x 2000 115 / 86, 5000 x 4000 80 / 62, 30000 x 4096 367 / 300, with longer rows 4000 x
// 5900 87 / 87.
bool strips_one_ok(int axis, int64_t nvec, int64_t veclen) {
  if (veclen <= 0 || nvec >= (1 << 24)) return false;
  if (axis == SRQ_AXIS_ROW) return veclen <= 4096 || strips_ok(nvec, 0, veclen);
  return veclen <= 2048 || (veclen <= 4096 && nvec * veclen <= 8200000);
}
// (Every workgroup adds up the counts before its vectors: scan and scatter in launches of their own / here, us:
// 8000 x 200 x 2000 94.9 / 82.3, 16000 x 200 x 200 66.2 / 61.8, 40 x 40000 x 1000 202 / 220, 60000 x 60 x 2000 505 / 539.)
bool strips_compact_ok(int64_t M, int64_t N) { return M <= kStripsMaxScan && N <= kStripsMaxScan; }

// (Rows per thread, calls at 5 % kept, us, 16 in 256 threads / 8 in 512: 512 x 512 x 1100 42 / 38, 1024 x 1024 x 2048 52 / 49,
// 300 x 3000 x 2048 67 / 65, 4096 x 4096 x 2048 228 / 234, 10000 x 1024 x 2048 249 / 256.  One step further either way loses:
// 4 in 512 threads at 2048 x 2048 x 1000 73 against 68, 8 in 1024 threads at 2048 x 2048 x 3000 143 against 134.)
#define SRQ_STRIPS_AS(TH, RT, NV4, CG, RPT, KERN, ROWS, ...)                                                                  \
  hipLaunchKernelGGL((KERN<TH, RT, NV4, CG, RPT>), dim3((unsigned)(strips + ((ROWS) + TH / RT - 1) / (TH / RT))), dim3(TH), 0, st, __VA_ARGS__)
#define SRQ_STRIPS(KERN, ROWS, ...)                                                                                       \
  do {                                                                                                              \
    const int strips = (int)((N + 4 * strip_cg(K) - 1) / (4 * strip_cg(K)));                                        \
    if (K <= 256) SRQ_STRIPS_AS(256, 64, 1, 4, 4, KERN, ROWS, __VA_ARGS__);                                          \
    else if (K <= 512) SRQ_STRIPS_AS(256, 64, 2, 4, 8, KERN, ROWS, __VA_ARGS__);                                     \
    else if (K <= 1024) SRQ_STRIPS_AS(256, 64, 4, 2, 8, KERN, ROWS, __VA_ARGS__);                                    \
    else if (K <= 2048 && N + (ROWS) <= 6000) SRQ_STRIPS_AS(512, 64, 8, 2, 8, KERN, ROWS, __VA_ARGS__);              \
    else if (K <= 2048) SRQ_STRIPS_AS(256, 64, 8, 2, 16, KERN, ROWS, __VA_ARGS__);                                   \
    else if (K <= 4096) SRQ_STRIPS_AS(512, 64, 16, 2, 16, KERN, ROWS, __VA_ARGS__);                                  \
    else SRQ_STRIPS_AS(512, 512, 4, 1, 16, KERN, ROWS, __VA_ARGS__);                                                 \
  } while (0)

hipError_t launch_quant_pair(const StripOperand& a, const StripOperand& b, int64_t M, int64_t N, int64_t K, int64_t Kc, int qmax,
                             int trunc, hipStream_t st) {
  SRQ_STRIPS(quant_pair_kernel, M, a, b, M, N, (int)K, (int)Kc, strips, (float)qmax, trunc);
  return hipGetLastError();
}

hipError_t launch_select_pair(const StripSelect& a, const StripSelect& b, int64_t M, int64_t N, int64_t K, hipStream_t st) {
  SRQ_STRIPS(select_pair_kernel, M, a, b, M, N, (int)K, strips);
  return hipGetLastError();
}

hipError_t launch_quant_strips(const StripOperand& s, int64_t N, int64_t K, int64_t ldq, int qmax, int trunc, hipStream_t st) {
  SRQ_STRIPS(quant_cols_kernel, 0, s, N, (int)K, ldq, strips, (float)qmax, trunc);
  return hipGetLastError();
}

hipError_t launch_reduce_cols(const StripReduce& s, int64_t N, int64_t K, int64_t Kc, int qmax, int trunc, hipStream_t st) {
  SRQ_STRIPS(reduce_cols_kernel, 0, s, N, (int)K, (int)Kc, strips, (float)qmax, trunc);
  return hipGetLastError();
}
#undef SRQ_STRIPS
#undef SRQ_STRIPS_AS

hipError_t launch_reduce_rows(const StripReduce& s, int64_t M, int64_t K, int64_t Kc, int qmax, int trunc, hipStream_t st) {
  const dim3 grid((unsigned)M);
  const float qm = (float)qmax;
  if (K <= 1024) hipLaunchKernelGGL((reduce_rows_kernel<256, 1>), grid, dim3(256), 0, st, s, (int)K, (int)Kc, qm, trunc);
  else if (K <= 2048) hipLaunchKernelGGL((reduce_rows_kernel<256, 2>), grid, dim3(256), 0, st, s, (int)K, (int)Kc, qm, trunc);
  else if (K <= 4096) hipLaunchKernelGGL((reduce_rows_kernel<256, 4>), grid, dim3(256), 0, st, s, (int)K, (int)Kc, qm, trunc);
  else hipLaunchKernelGGL((reduce_rows_kernel<512, 4>), grid, dim3(512), 0, st, s, (int)K, (int)Kc, qm, trunc);
  return hipGetLastError();
}

hipError_t launch_compact_pair(const StripCompact& a, const StripCompact& b, int64_t K, int64_t Kc, hipStream_t st) {
  if (a.nvec + b.nvec == 0) return hipSuccess;
#define SRQ_COMPACT(NV)                                                                                                    \
  do {                                                                                                                      \
    const int ga = (a.nvec + 3) / 4, gb = (b.nvec + 3) / 4;                                                                  \
    hipLaunchKernelGGL(compact_pair_kernel<NV>, dim3((unsigned)(ga + gb)), dim3(256), 0, st, a, b, ga, (int)K, (int)Kc);     \
  } while (0)
  if (Kc <= 1024) SRQ_COMPACT(1);
  else if (Kc <= 2048) SRQ_COMPACT(2);
  else if (Kc <= 4096) SRQ_COMPACT(4);
  else SRQ_COMPACT(8);
#undef SRQ_COMPACT
  return hipGetLastError();
}

}  // namespace srq
