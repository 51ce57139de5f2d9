// Which tiles a product is cut into, by rounds of tiles over the compute units.  Plain arithmetic, also compiled for
// the host by its test.
#ifndef SRQ_GEMM_ROUNDS_H_
#define SRQ_GEMM_ROUNDS_H_
#include <cstdint>

namespace srq {

// The compute units a product is cut up for.  Products with sums of |D_F| are always cut up for a whole device: the order
// of the additions, and by it means and thresholds, then depends on the shape alone, also on a part of a device.
constexpr int64_t kWholeDevice = 256;
inline int64_t cut_for(bool sums, int64_t device_cus) { return sums ? kWholeDevice : device_cus; }

// Rounds of bm x bn tiles over the compute units, and whether they would be nearly full
inline int64_t tile_rounds(int64_t M, int64_t N, int64_t bm, int64_t bn, int64_t cus) {
  return (((M + bm - 1) / bm) * ((N + bn - 1) / bn) + cus - 1) / cus;
}
inline bool fills_rounds(int64_t M, int64_t N, int64_t bm, int64_t bn, int64_t cus) {
  return 100 * ((M + bm - 1) / bm) * ((N + bn - 1) / bn) >= 85 * cus * tile_rounds(M, N, bm, bn, cus);
}

// The persistent kernel with 256 x 256 tiles or the one with smaller tiles?  In rounds of 256 x 128 tiles over the compute
// units; a round of 128 x 128 counts 4/7.  Against two of them a round of the persistent kernel, which stores a tile
// while it multiplies the next and loads less, takes for
//   one product          1 / 1.2: us, persistent / smaller tiles, 4096^2 x 512 25.7 / 31.6, 4096^3 62 / 75, 8192^3 403 / 485
//   a pair of products   1 / (0.96 + K / 40000), because the smaller tiles read and write C once for both:
//                        4096^2 x 512 63 / 58, 8192^2 x 1024 268 / 255, 4096^2 x 2048 89 / 91, 4096^3 127 / 139,
//                        8192^3 786 / 886; at most 1 / 1.4: as many rounds of tiles twice as large never pay.  Calls, ms:
//                        one round of either 2816^2 x 24064 1.38 / 1.25, x 40064 2.25 / 2.04; two against three 6144 x
//                        4096 x 10240 0.96 / 0.94, x 24064 2.73 / 2.77, 5120 x 4096 x 10240 0.92 / 0.89, x 24064 2.57 / 2.79
// and a last round that is less than half full counts half as much with tiles half as large (pairs): 6144 x 4096 x 8192
// 366 / 331, 4096 x 14336 x 4096 460 / 442; 2048 x 4096 x 4096 (half a round) 102 / 70.
inline bool large_tiles(int64_t M, int64_t N, int64_t K, bool pair, int64_t cus) {
  const double tall = (double)tile_rounds(M, N, 256, 128, cus), low = (double)tile_rounds(M, N, 128, 128, cus) * 4 / 7;
  const double slower = !pair ? 1.2 : K < 17600 ? 0.96 + (double)K / 40000 : 1.4;
  return slower * (low < tall ? low : tall) >= 2 * (double)tile_rounds(M, N, 256, 256, cus);
}

// 256 x 128 tiles rather than 128 x 128?  A compute unit takes about 1.75 times as long for one.  Calls at 5 % kept, us,
// 128 / 256: one round of 256 instead of two of 128, 2048 x 4096 x 2048 127 / 113, 2000 x 2100 x 2048 124 / 108; two instead of
// four, 4096 x 3328 x 1024 122 / 109; but two instead of three, 3072^2 x 1024 96 / 103.  (K-tiles of 0.43 and 0.8 us on every
// compute unit: 128-wide tiles are bound by the 20 clocks that the vector-memory path takes for a load, 640 and 960 of them
// for each K-tile against 512 and 1024 of matrix-core time.)
inline bool tall_tiles(int64_t M, int64_t N, int64_t cus) {
  return 7 * tile_rounds(M, N, 256, 128, cus) < 4 * tile_rounds(M, N, 128, 128, cus);
}

}  // namespace srq

#endif  // SRQ_GEMM_ROUNDS_H_
