"""The K-tiles that the matrix-core kernels load (csrc/gemm_ktiles.h, compiled here for the host): every
K-tile lies inside its row, and every byte of K is multiplied exactly once."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_06924_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "gemm_ktiles.h"
int main() {
  for (int K = 64; K <= 2048; K += 64)
    for (int kt = 0, nk = (K + srq::kKTile - 1) / srq::kKTile; kt < nk; ++kt)
      std::printf("%d %d %d %d %d\n", K, kt, srq::ktile_start(kt, K), kt == nk - 1 ? srq::last_ktile_mask(K, 0) : -1,
                  kt == nk - 1 ? srq::last_ktile_mask(K, 1) : -1);
  for (int K = 192; K <= 2048; K += 64)   // the persistent kernel: negative K
    for (int kt = 0, at = 0, nk = (K + srq::kKTile - 1) / srq::kKTile; kt < nk; ++kt) {
      std::printf("%d %d %d %d %d\n", -K, kt, at, -1, kt == 0 && (K & 64) ? 0 : -1);
      at += kt == 0 ? srq::first_ktile_step(K) : srq::kKTile;
    }
}
"""


def test_every_ktile_stays_in_its_row_and_counts_once(tmp_path):
    src, exe = tmp_path / "ktiles.cpp", tmp_path / "ktiles"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    rows = [tuple(map(int, ln.split())) for ln in subprocess.run([str(exe)], check=True, capture_output=True,
                                                                 text=True).stdout.splitlines()]
    for K in list(range(64, 2049, 64)) + list(range(-2048, -191, 64)):
        tiles = [r for r in rows if r[0] == K]
        K = abs(K)
        assert [r[1] for r in tiles] == list(range((K + 127) // 128))
        counted = []
        for _, _, start, head, tail in tiles:
            # (the one K-tile of K = 64 ends 64 bytes past the row: that end is in the lane's own offset, which
            # the descriptor's range check covers)
            assert start >= 0 and start % 16 == 0 and (start + 128 <= K or K == 64)
            counted += [start + 64 * h for h, m in ((0, head), (1, tail)) if m]
            assert head in (0, -1) and tail in (0, -1)
        assert sorted(counted) == list(range(0, K, 64))


CURSOR = r"""
#include <cstdio>
#include "gemm_ktiles.h"
int main() {
  for (int K = 64; K <= 2048; K += 64)
    for (int first = 0; first < 2; ++first)
      for (int last = first; last < 2; ++last) {
        const int nk = (K + srq::kKTile - 1) / srq::kKTile;
        srq::KtileCursor c = {first, 0};
        int step = -1;                       // 0: same rows, 1: the next product, 2: nothing is left
        for (int g = 0; g < nk * (last - first + 1) + 5; ++g) {
          std::printf("%d %d %d %d %d %d\n", K, first, last, step, c.prod, c.start(nk, K));
          step = c.same_rows(nk) ? 0 : c.next_product(nk, last) ? 1 : 2;
        }
      }
}
"""


def test_fetches_behind_the_last_ktile_are_at_offset_zero(tmp_path):
    """The stream of K-tiles of one or two products: each once, in order; then descriptors of no bytes (step 2), and no
    offset that a range check against their size less the offset would wrap around with."""
    src, exe = tmp_path / "cursor.cpp", tmp_path / "cursor"
    src.write_text(CURSOR)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    rows = [tuple(map(int, ln.split())) for ln in subprocess.run([str(exe)], check=True, capture_output=True,
                                                                 text=True).stdout.splitlines()]
    for K in range(64, 2049, 64):
        for first, last in ((0, 0), (0, 1), (1, 1)):
            got = [r[3:] for r in rows if r[:3] == (K, first, last)]
            starts = [min(128 * kt, max(K - 128, 0)) for kt in range((K + 127) // 128)]
            want = [(0 if kt else -1 if p == first else 1, p, at) for p in range(first, last + 1) for kt, at in enumerate(starts)]
            assert got[:len(want)] == want
            assert got[len(want):] == [(2, last, 0)] * 5
