// The epilogue of a 64 x 64 output tile of four waves (32 x 32 each, 2 x 2 blocks of 16 x 16), shared by the kernels
// that form one so that the sums of |D_F|, and with them the means and thresholds, are the same bits whichever ran.
#ifndef SRQ_GEMM_TILE64_H_
#define SRQ_GEMM_TILE64_H_
#include "gemm_lanes.h"

namespace srq {

// A wave's dequantized product added to `out` (add) or put there, in the layout of TileAccess<4>; with SUMS the sums of
// |D_F| of its 32 columns and 32 rows go to rowx[2][64] and colx[2][64], in double: the thresholds they become
// are then the same whatever kernel formed the product.  Columns: the 16 lanes' 8 values each end up one per
// pair of lanes (value rl >> 1).
template <bool SUMS>
static __device__ __forceinline__ void tile64_product(const v4i (&acc)[2][2], const float (&srow)[2], const v4f (&scol)[2], bool add,
                                                      v4f (&out)[4], int wm, int wn, int quad, int rl, double* rowx, double* colx) {
  double col8[8];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    v4f t[2];
    double r = 0.0;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        t[b][v] = (float)acc[a][b][v] * (srow[a] * scol[b][v]);
        if (SUMS) {
          const double d = (double)fabsf(t[b][v]);
          r += d;
          col8[4 * b + v] = a == 0 ? d : col8[4 * b + v] + d;
        }
      }
    if (SUMS) {
      r += __shfl_xor(r, 16, 64);
      r += __shfl_xor(r, 32, 64);
      if (quad == 0) rowx[wn * 64 + 32 * wm + 16 * a + rl] = r;
    }
    exchange_half_rows(t[0], t[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[2 * a + h][v] = add ? out[2 * a + h][v] + t[h][v] : t[h][v];
  }
  if (SUMS) {
    const double c = column_sum8(col8, rl);
    if (!(rl & 1)) colx[wm * 64 + 32 * wn + 16 * (rl >> 3) + 4 * quad + ((rl >> 1) & 3)] = c;
  }
}

// the tile's partial sums (behind a barrier after tile64_product), by the first two waves
static __device__ __forceinline__ void tile64_store_sums(const GemmEpilogue& ep, int tid, int64_t M, int64_t N, int tile_m, int tile_n,
                                                         uint32_t rows, uint32_t cols, const double* rowx, const double* colx) {
  if ((uint32_t)tid < rows) ep.row_part[(int64_t)tile_n * M + 64 * (int64_t)tile_m + tid] = rowx[tid] + rowx[64 + tid];
  if (tid >= 64 && (uint32_t)(tid - 64) < cols)
    ep.col_part[(int64_t)tile_m * N + 64 * (int64_t)tile_n + tid - 64] = colx[tid - 64] + colx[tid];
}

// alpha and beta
static __device__ __forceinline__ void tile64_scale(const GemmEpilogue& ep, bool has_beta, v4f (&out)[4], const v4f (&cin)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      out[i][v] = ep.alpha * out[i][v];
      if (has_beta) out[i][v] = out[i][v] + ep.beta * cin[i][v];
    }
}

}  // namespace srq

#endif  // SRQ_GEMM_TILE64_H_
