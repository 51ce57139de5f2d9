// Calls with an inner dimension of at most 256 and up to 1024 rows and columns: the whole of Algorithm 1 in two launches,
// where the kernels of strips.hip and gemm_tile64.hip take five (one instead of two without compensation).
//
//   short_first_kernel    a 64 x 64 tile of C per workgroup, from the FP32 operands: all of its 64 rows of A and 64
//                         columns of B fit the registers, so that it quantizes them itself (every tile of a row of
//                         tiles does so again), multiplies and leaves D_F and the partial sums of |D_F|.  The first
//                         workgroups of the grid take sixteen rows or columns each and write codes, residual codes
//                         and scales.
//   short_second_kernel   a tile of C per workgroup: thresholds from the partial sums, the reduced operands straight into
//                         LDS, both corrections, alpha and beta.  The first workgroups compact sixteen rows of A or
//                         columns of B each: means and thresholds, CSR / CSC.
//
// What bounds them: latency.  A launch that does nothing costs 3-4 us, a trip through a workgroup (operand loads, all in
// flight together, maxima, codes, LDS, products, C) as much again.  Hence loads without branches (one behind a
// branch is waited for before the next is issued: 15 us instead of 7 for the first launch at 256^3), few vector
// instructions per element (a wave's instruction takes four clocks: codes are rounded by an addition and packed by
// byte permutes, residuals are formed by the sixteen-vector workgroups alone), and no separate pass for anything.
// Calls at 5 % kept, us, separate launches / these: 256^3 23.3 / 14.1, 960 x 896 x 64 with beta 25.9 / 15.4, 100^3 23.3 /
// 12.8, 1024^2 x 128 25.1 / 16.7, 1024^2 x 256 25.9 / 18.4, 1000^2 x 250 27.7 / 25.4 (rows of A that are no multiple
// of 16 bytes are loaded by the element); 256^3 without compensation 10.9 / 8.0.  Larger ones would lose (2048^2 x
// 256 40.8 / 69 with 1024 tiles, that many times the quantization).
// The codes, the sums of |D_F| and the order in which they are added up are those of the other kernels (tile64_product;
// row_sum and col_sum), so that thresholds do not depend on the path taken.
#include "gemm_tile64.h"
#include "gemm_tiles.h"
#include "stream.h"
#include <type_traits>

namespace srq {
namespace {

constexpr int BT = 64, kTile = BT * kKTile;          // bytes of one K-tile of an operand tile in LDS
constexpr int kChunk = 16;                           // vectors a compacting workgroup takes

// LDS: K-tiles of 64 rows of 128 bytes, the 16-byte pieces of a row XOR-swizzled with (row >> 1) & 7
__device__ __forceinline__ int lds_at(int row, int e) {
  return (e >> 7) * kTile + row * kKTile + 16 * (((e & 127) >> 4) ^ ((row >> 1) & 7)) + (e & 15);
}

// maximum over the sixteen lanes of a row of lanes
__device__ __forceinline__ float max16(float m) {
  m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x128, 0xf, 0xf, true)));   // row_ror 8, 4, 2, 1
  m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x124, 0xf, 0xf, true)));
  m = fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x122, 0xf, 0xf, true)));
  return fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x121, 0xf, 0xf, true)));
}

__device__ __forceinline__ int left4(int n) { return n >= 4 ? 4 : n > 0 ? n : 0; }

// The first n (0 .. 4) of four values, zero for the others.  WHOLE: n is 0 or 4.
template <bool WHOLE>
__device__ __forceinline__ v4f load4(__amdgpu_buffer_rsrc_t r, uint32_t off, int n) {
  if (WHOLE) return buf_load_4(r, n > 0 ? off : kOutside, true);
  v4f x;
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] = buf_load_f32(r, v < n ? off + 4u * v : kOutside);
  return x;
}

// A lane's part of 64 rows of A: row 16 w + 4 g + lane / 16, elements 64 i + 4 (lane % 16) .. + 3
template <int KC>
struct RowsPatch {
  v4f x[4][KC / 64];
  __device__ __forceinline__ static int row(int g) { return 16 * (threadIdx.x >> 6) + 4 * g + ((threadIdx.x >> 4) & 3); }
  __device__ __forceinline__ static int elem(int i) { return 64 * i + 4 * (threadIdx.x & 15); }
  template <bool WHOLE>
  __device__ __forceinline__ void load_as(__amdgpu_buffer_rsrc_t r, uint32_t ldx, int rows, int K) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int i = 0; i < KC / 64; ++i)
        x[g][i] = load4<WHOLE>(r, 4u * ((uint32_t)row(g) * ldx + (uint32_t)elem(i)), row(g) < rows ? left4(K - elem(i)) : 0);
  }
  __device__ __forceinline__ void load(const float* X, int64_t ldx, int m0, int M, int K) {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(X + m0 * ldx, kRecords);
    if (K & 3) load_as<false>(r, (uint32_t)ldx, M - m0, K);
    else load_as<true>(r, (uint32_t)ldx, M - m0, K);
  }
};
// A lane's part of 64 columns of B: columns 4 (lane % 16) .. + 3, KC / 16 rows from k0() on
template <int KC>
struct ColsPatch {
  static constexpr int R = KC / 16;
  v4f x[R];
  __device__ __forceinline__ static int col() { return 4 * (threadIdx.x & 15); }
  __device__ __forceinline__ static int k0() { return R * (threadIdx.x >> 4); }
  template <bool WHOLE>
  __device__ __forceinline__ void load_as(__amdgpu_buffer_rsrc_t r, uint32_t ldx, int n, int K) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      x[i] = load4<WHOLE>(r, 4u * ((uint32_t)(k0() + i) * ldx + (uint32_t)col()), k0() + i < K ? n : 0);
  }
  __device__ __forceinline__ void load(const float* X, int64_t ldx, int n0, int N, int K) {
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(X + n0, kRecords);
    if (N & 3) load_as<false>(r, (uint32_t)ldx, left4(N - n0 - col()), K);
    else load_as<true>(r, (uint32_t)ldx, left4(N - n0 - col()), K);
  }
};

template <int R>
__device__ __forceinline__ void put_codes(int8_t* dst, const unsigned (&pk)[R / 4]) {   // R = 8 or 16 bytes, aligned to R
  if constexpr (R == 16) *reinterpret_cast<uint4*>(dst) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
  else *reinterpret_cast<uint2*>(dst) = make_uint2(pk[0], pk[1]);
}

// the four waves' 32 x 32 parts of the product of two operand tiles in LDS
template <int KC>
__device__ __forceinline__ void multiply(const int8_t* a, const int8_t* b, int wm, int wn, int quad, int rl, v4i (&acc)[2][2]) {
  const int key = (rl >> 1) & 7, a_row = (32 * wm + rl) * kKTile, b_row = (32 * wn + rl) * kKTile;
  const int xoff[2] = {16 * (quad ^ key), 16 * ((4 + quad) ^ key)};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4i{0, 0, 0, 0};
#pragma unroll
  for (int kt = 0; kt < KC / kKTile; ++kt)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      v4i fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fb[i] = *reinterpret_cast<const v4i*>(b + kt * kTile + b_row + xoff[s] + i * 16 * kKTile);
        fa[i] = *reinterpret_cast<const v4i*>(a + kt * kTile + a_row + xoff[s] + i * 16 * kKTile);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
}

// ---- quantization ----------------------------------------------------------------------------------
__device__ __forceinline__ float max_abs4(v4f x, float m) {
  return fmaxf(fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))), m);
}
__device__ __forceinline__ float quotient(float a, float b, bool ok) { return ok ? a / b : 0.f; }

struct ChunkShared {
  float t[kChunk];
  float red[2][4][kChunk];
  int count[kChunk];
  uint32_t wave[4][4];
  int64_t before[4];
  int chunk;
};

// sixteen rows of A, one sixteen lanes wide: codes, residual codes, scales
template <int KC, bool COMP, bool TRUNC>
__device__ __forceinline__ void quantize_rows(const ShortCall& g, int chunk) {
  constexpr int NI = KC / 64;
  const int tid = threadIdx.x, c = tid & 15, row = kChunk * chunk + (tid >> 4), K = g.K;
  const bool ok = row < g.M;
  v4f x[NI];
  const __amdgpu_buffer_rsrc_t rx = buf_rsrc(g.A + (int64_t)kChunk * chunk * g.lda, kRecords);
  auto load = [&](auto whole) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      x[i] = load4<decltype(whole)::value>(rx, 4u * ((uint32_t)(tid >> 4) * (uint32_t)g.lda + 64u * i + 4u * c), ok ? left4(K - 64 * i - 4 * c) : 0);
  };
  if (K & 3) load(std::false_type());
  else load(std::true_type());
  if (COMP && tid == 0) {                            // (what the second launch publishes there starts as absent)
    g.state_a[chunk] = -1;
    if (chunk == 0) *g.ticket = 0;
  }
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) m = max_abs4(x[i], m);
  const float amax = max16(m), qmax = g.qmax;
  const float lam = quotient(qmax, amax, amax > 0.f), sc = quotient(amax, qmax, amax > 0.f);
  unsigned pk[NI];
  float rm = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    v4f z;
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = biased_code(x[i][j], lam, qmax, TRUNC);
    const int n = left4(K - 64 * i - 4 * c);
    pk[i] = pack_codes(z[0], z[1], z[2], z[3], n);
    if (COMP) {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[i][j] = j < n ? x[i][j] - code_value(z[j]) * sc : 0.f;   // (0 * lam is not 0 where lam overflowed)
      rm = max_abs4(x[i], rm);
    }
  }
  if (!ok) return;
#pragma unroll
  for (int i = 0; i < NI; ++i) *reinterpret_cast<unsigned*>(g.Qa + (int64_t)row * KC + 64 * i + 4 * c) = pk[i];
  if (c == 0) { g.s_a[row] = sc; g.lam_a[row] = lam; }
  if (!COMP) return;
  const float ramax = max16(rm);                     // (a row's sixteen lanes are here or not together)
  const float rlam = quotient(qmax, ramax, ramax > 0.f);
  if (c == 0) g.s_ra[row] = quotient(ramax, qmax, ramax > 0.f);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    v4f z;
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = biased_code(x[i][j], rlam, qmax, TRUNC);
    *reinterpret_cast<unsigned*>(g.Ra + (int64_t)row * KC + 64 * i + 4 * c) = pack_codes(z[0], z[1], z[2], z[3], left4(K - 64 * i - 4 * c));
  }
}

// sixteen columns of B: four lanes wide, KC / 64 rows per thread
template <int KC, bool COMP, bool TRUNC>
__device__ __forceinline__ void quantize_cols(const ShortCall& g, int chunk, ChunkShared& sm) {
  constexpr int R = KC / 64;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, cg = tid & 3, row0 = R * (tid >> 2), v0 = kChunk * chunk, K = g.K;
  const int col = v0 + 4 * cg, ncol = left4(g.N - col);
  v4f x[R];
  const __amdgpu_buffer_rsrc_t rx = buf_rsrc(g.B + v0, kRecords);
  auto load = [&](auto whole) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      x[i] = load4<decltype(whole)::value>(rx, 4u * ((uint32_t)(row0 + i) * (uint32_t)g.ldb + 4u * (uint32_t)cg), row0 + i < K ? ncol : 0);
  };
  if (g.N & 3) load(std::false_type());
  else load(std::true_type());
  if (COMP && tid == 0) g.state_b[chunk] = -1;
  // a lane's four columns over the sixteen lanes of its kind, then over the waves
  auto col_max = [&](v4f m, int which) __attribute__((always_inline)) -> v4f {
#pragma unroll
    for (int off = 4; off < 64; off <<= 1)
#pragma unroll
      for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], __shfl_xor(m[c], off, 64));
    if (lane < 4) *reinterpret_cast<v4f*>(&sm.red[which][w][4 * cg]) = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const v4f r = *reinterpret_cast<const v4f*>(&sm.red[which][i][4 * cg]);
#pragma unroll
      for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], r[c]);
    }
    return m;
  };
  auto put = [&](int8_t* Q, const v4f (&z)[R]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const unsigned p = pack_codes(z[0][c], z[1][c], R == 4 ? z[R - 2][c] : kCodeBias, R == 4 ? z[R - 1][c] : kCodeBias, left4(K - row0));
      int8_t* dst = Q + (int64_t)(col + c) * KC + row0;
      if (c < ncol) {
        if (R == 4) *reinterpret_cast<unsigned*>(dst) = p;
        else *reinterpret_cast<unsigned short*>(dst) = (unsigned short)p;
      }
    }
  };
  v4f m = {0.f, 0.f, 0.f, 0.f}, rm = m;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], fabsf(x[i][c]));
  m = col_max(m, 0);
  const float qmax = g.qmax;
  v4f z[R];
  float lam[4], sc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lam[c] = quotient(qmax, m[c], m[c] > 0.f);
    sc[c] = quotient(m[c], qmax, m[c] > 0.f);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      z[i][c] = biased_code(x[i][c], lam[c], qmax, TRUNC);
      if (COMP) {
        x[i][c] = row0 + i < K ? x[i][c] - code_value(z[i][c]) * sc[c] : 0.f;
        rm[c] = fmaxf(rm[c], fabsf(x[i][c]));
      }
    }
  }
  put(g.Qb, z);
  if (tid < 4) { store_part(g.s_b + col, sc, ncol); store_part(g.lam_b + col, lam, ncol); }
  if (!COMP) return;
  rm = col_max(rm, 1);
  float rs[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float rlam = quotient(qmax, rm[c], rm[c] > 0.f);
    rs[c] = quotient(rm[c], qmax, rm[c] > 0.f);
#pragma unroll
    for (int i = 0; i < R; ++i) z[i][c] = biased_code(x[i][c], rlam, qmax, TRUNC);
  }
  put(g.Rb, z);
  if (tid < 4) store_part(g.s_rb + col, rs, ncol);
}

// ---- first launch ----------------------------------------------------------------------------------
template <int KC, bool COMP, bool TRUNC>
__global__ __launch_bounds__(256) void short_first_kernel(ShortCall g, int tiles_m, int tiles_n, int chunks_a, int chunks_b, GemmEpilogue ep) {
  constexpr int R = ColsPatch<KC>::R;
  __shared__ __attribute__((aligned(16))) int8_t ta[KC / kKTile * kTile], tb[KC / kKTile * kTile];
  __shared__ float red[4][BT], s_row[BT], s_col[BT];
  __shared__ double rowx[COMP ? 2 * BT : 1], colx[COMP ? 2 * BT : 1];
  __shared__ ChunkShared sm;
  const int bid = (int)blockIdx.x - chunks_a - chunks_b;
  if (bid < 0) {
    if ((int)blockIdx.x < chunks_a) quantize_rows<KC, COMP, TRUNC>(g, blockIdx.x);
    else quantize_cols<KC, COMP, TRUNC>(g, (int)blockIdx.x - chunks_a, sm);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
  const int quad = lane >> 4, rl = lane & 15, M = g.M, N = g.N, K = g.K;
  int tile_m, tile_n;
  tile_of(bid, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BT, n0 = tile_n * BT;
  RowsPatch<KC> a;
  ColsPatch<KC> b;
  b.load(g.B, g.ldb, n0, N, K);
  a.load(g.A, g.lda, m0, M, K);
  const uint32_t rows = (uint32_t)(M - m0 < BT ? M - m0 : BT), cols = (uint32_t)(N - n0 < BT ? N - n0 : BT);
  const TileAccess<4> tile = {32 * wm + (rl & 7), 32 * wn + 16 * (rl >> 3) + 4 * quad, rows, cols, rows == BT && cols == BT};
  v4f out[4], cin[4];
  const bool has_beta = !COMP && ep.final_scale && ep.beta != 0.f;
  if (has_beta) tile.load(cin, ep.Cin + (int64_t)m0 * ep.ldcin + n0, (uint32_t)ep.ldcin);
  const float qmax = g.qmax;

  // ---- maxima of the columns of B, on their way through LDS while the rows of A are quantized
  const int col = b.col(), k0 = b.k0();
  v4f m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], fabsf(b.x[i][c]));
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    m[c] = fmaxf(m[c], __shfl_xor(m[c], 16, 64));
    m[c] = fmaxf(m[c], __shfl_xor(m[c], 32, 64));
  }
  if (quad == 0) *reinterpret_cast<v4f*>(&red[w][4 * rl]) = m;
  // ---- rows of A
#pragma unroll
  for (int gr = 0; gr < 4; ++gr) {
    const int row = a.row(gr);
    float am = 0.f;
#pragma unroll
    for (int i = 0; i < KC / 64; ++i) am = max_abs4(a.x[gr][i], am);
    const float amax = max16(am), lam = quotient(qmax, amax, amax > 0.f);
#pragma unroll
    for (int i = 0; i < KC / 64; ++i) {
      v4f z;
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = biased_code(a.x[gr][i][j], lam, qmax, TRUNC);
      *reinterpret_cast<unsigned*>(ta + lds_at(row, a.elem(i))) = pack_codes(z[0], z[1], z[2], z[3], left4(K - a.elem(i)));
    }
    if (rl == 0) s_row[row] = quotient(amax, qmax, amax > 0.f);
  }
  __syncthreads();
  // ---- columns of B
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const v4f r = *reinterpret_cast<const v4f*>(&red[i][4 * rl]);
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], r[c]);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float lam = quotient(qmax, m[c], m[c] > 0.f);
    if (k0 == 0) s_col[col + c] = quotient(m[c], qmax, m[c] > 0.f);
    unsigned pk[R / 4];
#pragma unroll
    for (int i = 0; i < R; i += 4) {
      float z[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = biased_code(b.x[i + j][c], lam, qmax, TRUNC);
      pk[i / 4] = pack_codes(z[0], z[1], z[2], z[3], left4(K - k0 - i));
    }
    put_codes<R>(tb + lds_at(col + c, k0), pk);
  }
  __syncthreads();

  // ---- product
  v4i acc[2][2];
  multiply<KC>(ta, tb, wm, wn, quad, rl, acc);
  float srow[2];
  v4f scol[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    srow[i] = s_row[32 * wm + 16 * i + rl];
    scol[i] = *reinterpret_cast<const v4f*>(&s_col[32 * wn + 16 * i + 4 * quad]);
  }
  tile64_product<COMP>(acc, srow, scol, false, out, wm, wn, quad, rl, rowx, colx);
  if (COMP) {
    __syncthreads();
    tile64_store_sums(ep, tid, M, N, tile_m, tile_n, rows, cols, rowx, colx);
  } else if (ep.final_scale) {
    tile64_scale(ep, has_beta, out, cin);
  }
  tile.store(out, ep.C + (int64_t)m0 * ep.ldc + n0, (uint32_t)ep.ldc);
}

// ---- means ---------------------------------------------------------------------------------------
// Sums of the partial sums of one row / one column, added up as select_pair_kernel<256, 64, 1, 4, 4> of strips.hip does, which
// the other executions of such a call run: a row's as a tree over 64 lanes, distances 32, 16, ... 1 (absent ones are
// zero); a column's, sixteen at most, in pairs, pairs of pairs, and the four sums of four one after the other.
// (All loads at once, those of absent partials from the last one that exists: a load behind a branch is waited for
// before the next is issued.)
template <int LEAVES>
__device__ __forceinline__ void load_parts(double (&y)[LEAVES], const double* part, int64_t stride, int nparts) {
#pragma unroll
  for (int p = 0; p < LEAVES; ++p) y[p] = part[(p < nparts ? p : nparts - 1) * stride];
#pragma unroll
  for (int p = 0; p < LEAVES; ++p) y[p] = p < nparts ? y[p] : 0.0;
}
template <int LEAVES>
__device__ __forceinline__ double row_tree(const double* part, int64_t stride, int nparts) {
  double y[LEAVES];
  load_parts(y, part, stride, nparts);
#pragma unroll
  for (int h = LEAVES / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int p = 0; p < h; ++p) y[p] += y[p + h];
  return y[0];
}
template <int LEAVES>
__device__ __forceinline__ double col_tree(const double* part, int64_t stride, int nparts) {
  double y[LEAVES], all = 0.0;
  load_parts(y, part, stride, nparts);
#pragma unroll
  for (int w = 0; w < LEAVES / 4; ++w) all += (y[4 * w] + y[4 * w + 1]) + (y[4 * w + 2] + y[4 * w + 3]);
  return all;
}
__device__ __forceinline__ double row_sum(const double* part, int64_t stride, int nparts) {
  return nparts <= 4 ? row_tree<4>(part, stride, nparts) : row_tree<16>(part, stride, nparts);
}
__device__ __forceinline__ double col_sum(const double* part, int64_t stride, int nparts) {
  return nparts <= 4 ? col_tree<4>(part, stride, nparts) : col_tree<16>(part, stride, nparts);
}
__device__ __forceinline__ void threshold_a(const ShortCall& g, int row, float& mean, float& t) {
  mean = (float)(row_sum(g.row_part + row, g.M, (g.N + BT - 1) / BT) / (double)g.N);
  t = g.theta_a * mean;
}
__device__ __forceinline__ void threshold_b(const ShortCall& g, int col, float& mean, float& t) {
  mean = (float)(col_sum(g.col_part + col, g.N, (g.M + BT - 1) / BT) / (double)g.M);
  t = g.theta_b * mean;
}

// ---- compaction ------------------------------------------------------------------------------------
// The chunk a compacting workgroup takes: the next one in the order in which they start (one counter, rows of A before
// columns of B, whatever their indices in the grid are).
__device__ __forceinline__ int take_chunk(int32_t* ticket, int* sm) {
  if (threadIdx.x == 0) *sm = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*sm);
}
// Kept entries of the chunks before this one: every chunk publishes its own number as soon as it has it, before it waits,
// and waits for lower chunks only.  Those have been taken before, by workgroups that are running and wait for nothing
// until they have published: every wait ends, in whatever order and wherever workgroups are started and whatever else,
// calls on other streams among it, has taken the compute units.
__device__ __forceinline__ int64_t kept_before(int32_t* state, int chunk, int kept, int64_t* sm) {
  const int tid = threadIdx.x;
  if (tid == 0) __hip_atomic_store(state + chunk, kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int64_t sum = 0;
  for (int i = tid; i < chunk; i += 256) {
    int32_t k;
    while ((k = __hip_atomic_load(state + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < 0) __builtin_amdgcn_s_sleep(1);
    sum += k;
  }
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
  if ((tid & 63) == 0) sm[tid >> 6] = sum;
  __syncthreads();
  return sm[0] + sm[1] + sm[2] + sm[3];
}

__device__ __forceinline__ void put_entry(const ShortCompact& o, int64_t p, int e, int code) {
  if (p < o.capacity) { o.idx[p] = e; o.val[p] = (int8_t)code; }
}
__device__ __forceinline__ void put_ptr(const ShortCompact& o, const ChunkShared& sm, int v0, int nvec, int64_t first) {
  const int tid = threadIdx.x;
  if (tid < kChunk && v0 + tid < nvec) {
    int64_t p = first;
    for (int i = 0; i < tid; ++i) p += sm.count[i];
    o.ptr[v0 + tid] = (int32_t)p;
    if (v0 + tid == nvec - 1) {
      o.ptr[nvec] = (int32_t)(p + sm.count[tid]);
      *o.nnz = p + sm.count[tid];
    }
  }
}

// rows 16 chunk .. + 15 of A, one sixteen lanes wide
template <int KC>
__device__ __forceinline__ void compact_rows(const ShortCall& g, int chunk, ChunkShared& sm) {
  constexpr int NI = KC / 64;
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, r = tid >> 4, v0 = kChunk * chunk, M = g.M, K = g.K;
  const bool ok = g.term_a && v0 + r < M;
  v4f x[NI];
  unsigned code[NI];
  const __amdgpu_buffer_rsrc_t rx = buf_rsrc(g.A + v0 * g.lda, kRecords), rq = buf_rsrc(g.Qa + (int64_t)v0 * KC, kRecords);
  auto load = [&](auto whole) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = 64 * i + 4 * c;
      x[i] = load4<decltype(whole)::value>(rx, 4u * ((uint32_t)r * (uint32_t)g.lda + (uint32_t)e), ok ? left4(K - e) : 0);
      code[i] = __builtin_amdgcn_raw_buffer_load_b32(rq, ok ? r * KC + e : kOutside, 0, 0);
    }
  };
  if (K & 3) load(std::false_type());
  else load(std::true_type());
  if (tid < kChunk && v0 + tid < M) {
    float mean, t;
    threshold_a(g, v0 + tid, mean, t);
    sm.t[tid] = t;
    g.drow[v0 + tid] = mean;
    g.t_a[v0 + tid] = t;
  }
  __syncthreads();
  if (!g.term_a) return;                             // (the whole workgroup)
  const float t = sm.t[r];
  unsigned nib[NI];
  int at[NI], kept = 0;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    nib[i] = (fabsf(x[i].x) > t ? 1u : 0u) | (fabsf(x[i].y) > t ? 2u : 0u) | (fabsf(x[i].z) > t ? 4u : 0u) | (fabsf(x[i].w) > t ? 8u : 0u);
    nib[i] = ok ? nib[i] & ((1u << left4(K - 64 * i - 4 * c)) - 1u) : 0u;
    const int n = __popc(nib[i]);
    // (the row's sixteen lanes: bits 16 (lane / 16) .. of the ballots)
    const int sh = lane & 48;
    const uint32_t b0 = (uint32_t)(__ballot(n & 1) >> sh) & 0xffffu, b1 = (uint32_t)(__ballot(n & 2) >> sh) & 0xffffu,
                   b2 = (uint32_t)(__ballot(n & 4) >> sh) & 0xffffu, lower = (1u << c) - 1u;
    at[i] = kept + __popc(b0 & lower) + 2 * __popc(b1 & lower) + 4 * __popc(b2 & lower);
    kept += __popc(b0) + 2 * __popc(b1) + 4 * __popc(b2);
  }
  if (c == 0) sm.count[r] = kept;
  __syncthreads();
  int total = 0, mine = 0;
#pragma unroll
  for (int i = 0; i < kChunk; ++i) {
    total += sm.count[i];
    if (i < r) mine += sm.count[i];
  }
  const int64_t first = kept_before(g.state_a, chunk, total, sm.before);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    int64_t p = first + mine + at[i];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (nib[i] >> j & 1u) put_entry(g.ca, p++, 64 * i + 4 * c + j, (int)(code[i] >> (8 * j)));
  }
  put_ptr(g.ca, sm, v0, M, first);
}

// columns 16 chunk .. + 15 of B: four lanes wide, KC / 64 rows per thread
template <int KC>
__device__ __forceinline__ void compact_cols(const ShortCall& g, int chunk, ChunkShared& sm) {
  constexpr int R = KC / 64;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, cg = tid & 3, row0 = R * (tid >> 2), v0 = kChunk * chunk, N = g.N, K = g.K;
  const int ncol = g.term_b ? left4(N - v0 - 4 * cg) : 0;
  v4f x[R];
  unsigned code[4];
  const __amdgpu_buffer_rsrc_t rx = buf_rsrc(g.B + v0, kRecords), rq = buf_rsrc(g.Qb + (int64_t)v0 * KC, kRecords);
  auto load = [&](auto whole) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      x[i] = load4<decltype(whole)::value>(rx, 4u * ((uint32_t)(row0 + i) * (uint32_t)g.ldb + 4u * (uint32_t)cg), row0 + i < K ? ncol : 0);
  };
  if (N & 3) load(std::false_type());
  else load(std::true_type());
#pragma unroll
  for (int c = 0; c < 4; ++c) {                      // (R = 2: the dword of rows row0 .. or row0 - 2 ..)
    const uint32_t w4 = __builtin_amdgcn_raw_buffer_load_b32(rq, c < ncol ? (4 * cg + c) * KC + (row0 & ~3) : kOutside, 0, 0);
    code[c] = w4 >> (8 * (row0 & 3));
  }
  if (tid < kChunk && v0 + tid < N) {
    float mean, t;
    threshold_b(g, v0 + tid, mean, t);
    sm.t[tid] = t;
    g.dcol[v0 + tid] = mean;
    g.t_b[v0 + tid] = t;
  }
  __syncthreads();
  if (!g.term_b) return;                             // (the whole workgroup)
  // kept rows of a column: R bits; the four columns' counts in the bytes of a word (64 at most in a wave)
  unsigned bits[4] = {0, 0, 0, 0}, cnt = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float t = sm.t[4 * cg + c];
#pragma unroll
    for (int i = 0; i < R; ++i) bits[c] |= c < ncol && row0 + i < K && fabsf(x[i][c]) > t ? 1u << i : 0u;
    cnt |= (unsigned)__popc(bits[c]) << (8 * c);
  }
  unsigned incl = cnt;
#pragma unroll
  for (int off = 4; off < 64; off <<= 1) {
    const unsigned below = __shfl_up(incl, off, 64);
    if (lane >= off) incl += below;
  }
  if (lane >= 60) sm.wave[w][cg] = incl;
  __syncthreads();
  int at[4], total = 0, mine = 0, before[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    at[c] = (int)((incl - cnt) >> (8 * c) & 0xffu);
    for (int i = 0; i < w; ++i) at[c] += (int)(sm.wave[i][cg] >> (8 * c) & 0xffu);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      int n = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) n += (int)(sm.wave[i][q] >> (8 * c) & 0xffu);
      if (q == cg) before[c] = mine;
      if (q <= cg) mine += n;
      total += n;
      if (tid == 0) sm.count[4 * q + c] = n;
    }
  const int64_t first = kept_before(g.state_b, chunk, total, sm.before);   // (its barrier publishes the counts)
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int64_t p = first + before[c] + at[c];
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (bits[c] >> i & 1u) put_entry(g.cb, p++, row0 + i, (int)(code[c] >> (8 * i)));
  }
  put_ptr(g.cb, sm, v0, N, first);
}

// ---- second launch ---------------------------------------------------------------------------------
template <int KC>
__global__ __launch_bounds__(256) void short_second_kernel(ShortCall g, int tiles_m, int tiles_n, int chunks_a, int chunks_b, GemmEpilogue ep) {
  constexpr int kOperand = KC / kKTile * kTile, R = ColsPatch<KC>::R;
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];       // A', RB, RA, B'
  __shared__ ChunkShared sm;
  __shared__ float t_row[BT], t_col[BT];
  if ((int)blockIdx.x < chunks_a + chunks_b) {
    const int chunk = take_chunk(g.ticket, &sm.chunk);
    if (chunk < chunks_a) return compact_rows<KC>(g, chunk, sm);
    return compact_cols<KC>(g, chunk - chunks_a, sm);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) int8_t*)lds);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
  const int quad = lane >> 4, rl = lane & 15, M = g.M, N = g.N, K = g.K;
  int tile_m, tile_n;
  tile_of((int)blockIdx.x - chunks_a - chunks_b, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BT, n0 = tile_n * BT;
  const uint32_t rows = (uint32_t)(M - m0 < BT ? M - m0 : BT), cols = (uint32_t)(N - n0 < BT ? N - n0 : BT);

  // ---- residual codes straight into LDS: wave w fetches rows 16 w .. + 15, eight per load; rows past the end read as zero
  auto fetch = [&](const int8_t* Q, uint32_t n, int slot) __attribute__((always_inline)) {
    const uint64_t base = (uint64_t)(uintptr_t)Q;
    const v4i rsrc = {(int)(uint32_t)base, (int)(uint32_t)(base >> 32), (int)(n * KC), 0x00020000};
#pragma unroll
    for (int kt = 0; kt < KC / kKTile; ++kt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t row = 16 * w + 8 * j + (lane >> 3), voff = row * KC + kt * kKTile + 16 * ((lane & 7) ^ ((row >> 1) & 7));
        const uint32_t dst = lds0 + slot * kOperand + kt * kTile + (16 * w + 8 * j) * kKTile;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(voff), "s"(rsrc) : "memory", "m0");
      }
  };
  if (g.term_a) fetch(g.Rb + (int64_t)n0 * KC, cols, 1);
  if (g.term_b) fetch(g.Ra + (int64_t)m0 * KC, rows, 2);
  RowsPatch<KC> a;
  ColsPatch<KC> b;
  unsigned ca[4][KC / 64], cb[4][R / 4];
  const int col = b.col(), k0 = b.k0();
  if (g.term_a) {
    a.load(g.A, g.lda, m0, M, K);
    const __amdgpu_buffer_rsrc_t rqa = buf_rsrc(g.Qa + (int64_t)m0 * KC, rows * KC);   // (rows past the end read as zero)
#pragma unroll
    for (int gr = 0; gr < 4; ++gr)
#pragma unroll
      for (int i = 0; i < KC / 64; ++i)
        ca[gr][i] = __builtin_amdgcn_raw_buffer_load_b32(rqa, a.row(gr) * KC + a.elem(i), 0, 0);
  }
  if (g.term_b) {
    b.load(g.B, g.ldb, n0, N, K);
    const __amdgpu_buffer_rsrc_t rqb = buf_rsrc(g.Qb + (int64_t)n0 * KC, cols * KC);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < R / 4; ++i) cb[c][i] = __builtin_amdgcn_raw_buffer_load_b32(rqb, (col + c) * KC + k0 + 4 * i, 0, 0);
  }
  const TileAccess<4> tile = {32 * wm + (rl & 7), 32 * wn + 16 * (rl >> 3) + 4 * quad, rows, cols, rows == BT && cols == BT};
  v4f out[4], cin[4];
  const bool has_beta = ep.final_scale && ep.beta != 0.f;
  tile.load(out, ep.C + (int64_t)m0 * ep.ldc + n0, (uint32_t)ep.ldc);
  if (has_beta) tile.load(cin, ep.Cin + (int64_t)m0 * ep.ldcin + n0, (uint32_t)ep.ldcin);
  float mean, t = 0.f;
  if (w == 0) {
    if (lane < (int)rows) threshold_a(g, m0 + lane, mean, t);
    t_row[lane] = t;
  } else if (w == 1) {
    if (lane < (int)cols) threshold_b(g, n0 + lane, mean, t);
    t_col[lane] = t;
  }
  __syncthreads();

  // ---- the reduced operands (places past K have zero codes)
  if (g.term_a) {
#pragma unroll
    for (int gr = 0; gr < 4; ++gr) {
      const float th = t_row[a.row(gr)];
#pragma unroll
      for (int i = 0; i < KC / 64; ++i) {
        unsigned keep = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) keep |= fabsf(a.x[gr][i][j]) > th ? 0xffu << (8 * j) : 0u;
        *reinterpret_cast<unsigned*>(lds + lds_at(a.row(gr), a.elem(i))) = ca[gr][i] & keep;
      }
    }
  }
  if (g.term_b) {
    const v4f t4 = *reinterpret_cast<const v4f*>(&t_col[col]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      unsigned pk[R / 4];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if ((i & 3) == 0) pk[i >> 2] = 0;
        pk[i >> 2] |= fabsf(b.x[i][c]) > t4[c] ? 0xffu << (8 * (i & 3)) : 0u;
      }
#pragma unroll
      for (int i = 0; i < R / 4; ++i) pk[i] &= cb[c][i];
      put_codes<R>(lds + 3 * kOperand + lds_at(col + c, k0), pk);
    }
  }
  wait_loads();
  __syncthreads();

  // ---- both corrections, in the order of Algorithm 1
  const uint32_t ra = 4u * rows, rb = 4u * cols;
  auto correct = [&](int slot, const float* s_row, const float* s_col) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsr = buf_rsrc(s_row + m0, ra), rsc = buf_rsrc(s_col + n0, rb);
    float srow[2];
    v4f scol[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      srow[i] = buf_load_f32(rsr, 4u * (uint32_t)(32 * wm + 16 * i + rl));
      scol[i] = buf_load_4(rsc, 4u * (uint32_t)(32 * wn + 16 * i + 4 * quad), tile.full);
    }
    v4i acc[2][2];
    multiply<KC>(lds + slot * kOperand, lds + (slot + 1) * kOperand, wm, wn, quad, rl, acc);
    tile64_product<false>(acc, srow, scol, true, out, wm, wn, quad, rl, nullptr, nullptr);
  };
  if (g.term_a) correct(0, g.s_a, g.s_rb);
  if (g.term_b) correct(2, g.s_ra, g.s_b);
  if (ep.final_scale) tile64_scale(ep, has_beta, out, cin);
  tile.store(out, ep.C + (int64_t)m0 * ep.ldc + n0, (uint32_t)ep.ldc);
}

}  // namespace

bool short_ok(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, const GemmEpilogue& ep) {
  if (M <= 0 || N <= 0 || K <= 0 || K > 256 || M > 16 * BT || N > 16 * BT) return false;   // (sixteen partial sums)
  if (lda >= (1 << 22) || ldb >= (1 << 20)) return false;    // 32-bit byte offsets within 64 rows of A, 256 of B
  return ep.ldc < (1 << 22) && !(ep.final_scale && ep.beta != 0.f && ep.ldcin >= (1 << 22));
}

hipError_t launch_short_first(const ShortCall& g, bool comp, const GemmEpilogue& ep, hipStream_t st) {
  const int tm = (g.M + BT - 1) / BT, tn = (g.N + BT - 1) / BT, ca = (g.M + kChunk - 1) / kChunk, cb = (g.N + kChunk - 1) / kChunk;
  const dim3 grid((unsigned)(ca + cb + tm * tn));
  void (*kern)(ShortCall, int, int, int, int, GemmEpilogue);
#define SRQ_FIRST(KC, COMP) kern = g.trunc ? short_first_kernel<KC, COMP, true> : short_first_kernel<KC, COMP, false>
  if (g.K <= 128) { if (comp) SRQ_FIRST(128, true); else SRQ_FIRST(128, false); }
  else { if (comp) SRQ_FIRST(256, true); else SRQ_FIRST(256, false); }
#undef SRQ_FIRST
  hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, g, tm, tn, ca, cb, ep);
  return hipGetLastError();
}

hipError_t launch_short_second(const ShortCall& g, const GemmEpilogue& ep, hipStream_t st) {
  const int tm = (g.M + BT - 1) / BT, tn = (g.N + BT - 1) / BT, ca = (g.M + kChunk - 1) / kChunk, cb = (g.N + kChunk - 1) / kChunk;
  const int bytes = 4 * (g.K <= 128 ? 1 : 2) * kTile;
  auto kern = g.K <= 128 ? short_second_kernel<128> : short_second_kernel<256>;
  if (bytes > 48 * 1024) {
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(ca + cb + tm * tn)), dim3(256), bytes, st, g, tm, tn, ca, cb, ep);
  return hipGetLastError();
}

}  // namespace srq
