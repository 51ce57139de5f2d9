// K-tiles of the matrix-core kernels that load 128 bytes of every row at a time (K a multiple of 64): plain
// arithmetic, also compiled for the host by its test.
#ifndef SRQ_GEMM_KTILES_H_
#define SRQ_GEMM_KTILES_H_

#ifdef __HIPCC__
#define SRQ_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SRQ_HOST_DEVICE inline
#endif

namespace srq {

constexpr int kKTile = 128;

// First byte of K-tile kt.  Where K is an odd multiple of 64 the last K-tile is the row's last 128 bytes: of
// its two halves the first has been multiplied before and is masked.  So no load leaves its row, whether or
// not the hardware counts the scalar offset into the range check of the descriptor.  (K = 64 has one K-tile,
// at 0; its second half is masked, and where the last row of the operand ends the descriptor does.)
static SRQ_HOST_DEVICE int ktile_start(int kt, int K) {
  const int at = kt * kKTile, last = K < kKTile ? 0 : K - kKTile;
  return at < last ? at : last;
}
// mask for the fragments of half `half` (0, 1) of the last K-tile: all ones if its products count
static SRQ_HOST_DEVICE int last_ktile_mask(int K, int half) {
  return (K & 64) && half == (K < kKTile ? 1 : 0) ? 0 : -1;
}

// The persistent kernel (K > 128) has the half K-tile in front: its first K-tile counts for its first 64 where K
// is an odd multiple of 64, the second starts there and the last ends with the row.  (Masked at the end, the
// fragments are one kept register too many in the kernel without sums, which then spills inside the K loop:
// 8192^3, random codes, 433 us against 388.)
static SRQ_HOST_DEVICE int first_ktile_step(int K) { return kKTile - (K & 64); }

// Where a kernel is that fetches ahead of the K-tiles it multiplies, of products `prod` .. last, and goes on issuing its
// loads when none is left: then with descriptors of no bytes and at offset zero.  (The range check may be against the
// size less the scalar offset, which for no bytes and an offset is a large number.)
struct KtileCursor {
  int prod, kt;                                      // kt: from the number of K-tiles on nothing is left
  SRQ_HOST_DEVICE bool same_rows(int nk) {           // to the next K-tile of the product
    if (kt + 1 >= nk) return false;
    ++kt;
    return true;
  }
  SRQ_HOST_DEVICE bool next_product(int nk, int last) {   // ... or of the next one
    if (prod >= last) {
      kt = nk;
      return false;
    }
    ++prod;
    kt = 0;
    return true;
  }
  SRQ_HOST_DEVICE int start(int nk, int K) const { return kt < nk ? ktile_start(kt, K) : 0; }
};

}  // namespace srq

#undef SRQ_HOST_DEVICE
#endif  // SRQ_GEMM_KTILES_H_
