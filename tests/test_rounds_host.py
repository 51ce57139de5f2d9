"""The rule between tiles of 256 x 256 and smaller ones (csrc/gemm_rounds.h, compiled here for the host)."""
import os
import random
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_06924_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "gemm_rounds.h"
int main() {
  long long M, N, K, cus;
  while (std::scanf("%lld %lld %lld %lld", &M, &N, &K, &cus) == 4)
    std::printf("%d %d\n", srq::large_tiles(M, N, K, false, cus), srq::large_tiles(M, N, K, true, cus));
}
"""


def test_as_many_rounds_of_twice_as_large_tiles_are_never_taken(tmp_path):
    """However long K is: 2816 x 2816 in 256 x 256 tiles leaves half of the compute units idle in the one round that tiles
    of 256 x 128 need as well."""
    src, exe = tmp_path / "rounds.cpp", tmp_path / "rounds"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    rng = random.Random(5)
    # one round of either tiles; two of 256 x 256 against three of 256 x 128; one against two
    shapes = [(2816, 2816, 42048, 256), (2816, 2816, 133120, 256), (6144, 4096, 8192, 256), (6144, 4096, 24064, 256),
              (4096, 4096, 512, 256), (4096, 4096, 4096, 256)]
    shapes += [(rng.randint(1, 20000), rng.randint(1, 20000), 64 * rng.randint(3, 2080), rng.choice((32, 64, 256))) for _ in range(3000)]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, s)) for s in shapes), check=True, capture_output=True,
                         text=True).stdout.split()
    one, pair = [x == "1" for x in out[::2]], [x == "1" for x in out[1::2]]
    assert len(pair) == len(shapes)
    assert one[:6] == [False, False, False, False, True, True]
    assert pair[:6] == [False, False, False, True, False, True]
    for (M, N, K, cus), a, p in zip(shapes, one, pair):
        rounds = [-(-(-(-M // 256) * -(-N // n)) // cus) for n in (256, 128)]
        assert rounds[0] < rounds[1] or not (a or p), (M, N, K, cus)
