"""The rules between tiles of 256 x 256, 256 x 128 and 128 x 128 (csrc/gemm_rounds.h, compiled here for the host)."""
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
    std::printf("%d %d %d %d\n", srq::large_tiles(M, N, K, false, cus), srq::large_tiles(M, N, K, true, cus),
                srq::large_tiles(M, N, K, false, srq::cut_for(true, cus)), srq::tall_tiles(M, N, srq::cut_for(true, cus)));
}
"""


def decisions(tmp_path, shapes):
    """One product and a pair without sums in large tiles; with sums: large tiles, tall ones among the smaller."""
    src, exe = tmp_path / "rounds.cpp", tmp_path / "rounds"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, s)) for s in shapes), check=True, capture_output=True,
                         text=True).stdout.splitlines()
    assert len(out) == len(shapes)
    return [[x == "1" for x in ln.split()] for ln in out]


def test_products_with_sums_are_cut_by_the_shape_alone(tmp_path):
    """The same tiles, hence the same order of the additions, on a whole device and on parts of one."""
    rng = random.Random(6)
    shapes = [(rng.randint(1, 12000), rng.randint(1, 12000), 64 * rng.randint(3, 200)) for _ in range(500)]
    got = [decisions(tmp_path, [(*s, cus) for s in shapes]) for cus in (256, 128, 64, 32)]
    assert all([d[2:] for d in g] == [d[2:] for d in got[0]] for g in got[1:])
    assert any(d[2] for d in got[0]) and any(d[3] for d in got[0]) and got[0] != got[3]


def test_as_many_rounds_of_twice_as_large_tiles_are_never_taken(tmp_path):
    """However long K is: 2816 x 2816 in 256 x 256 tiles leaves half of the compute units idle in the one round that tiles
    of 256 x 128 need as well."""
    rng = random.Random(5)
    # one round of either tiles; two of 256 x 256 against three of 256 x 128; one against two
    shapes = [(2816, 2816, 42048, 256), (2816, 2816, 133120, 256), (6144, 4096, 8192, 256), (6144, 4096, 24064, 256),
              (4096, 4096, 512, 256), (4096, 4096, 4096, 256)]
    shapes += [(rng.randint(1, 20000), rng.randint(1, 20000), 64 * rng.randint(3, 2080), rng.choice((32, 64, 256))) for _ in range(3000)]
    one, pair = zip(*(d[:2] for d in decisions(tmp_path, shapes)))
    assert one[:6] == (False, False, False, False, True, True)
    assert pair[:6] == (False, False, False, True, False, True)
    for (M, N, K, cus), a, p in zip(shapes, one, pair):
        rounds = [-(-(-(-M // 256) * -(-N // n)) // cus) for n in (256, 128)]
        assert rounds[0] < rounds[1] or not (a or p), (M, N, K, cus)
