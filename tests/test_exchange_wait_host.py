"""The wait of workgroups for each other's words (csrc/exchange_wait.h, compiled here for the host, with a clock of its own)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_06924_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "exchange_wait.h"
int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) std::printf("%u ", srq::exchange_ticks(argv[i]));
  if (argc > 1) return std::printf("%u\n", srq::exchange_ticks(nullptr)), 0;
  // ticks, words, and when each of them is published (negative: never)
  long long ticks, n, at;
  while (std::scanf("%lld %lld", &ticks, &n) == 2) {
    srq::ExchangeWait wait{(uint32_t)ticks};
    uint64_t time = 1000;       // a look at a word takes one tick, a pause three
    int found = 0;
    for (int i = 0; i < n && std::scanf("%lld", &at) == 1; ++i)
      found += wait.word([&]() { ++time; return (uint32_t)(at >= 0 && time >= 1000 + (uint64_t)at); }, [](uint32_t w) { return w != 0; },
                         [&]() { return time; }, [&]() { time += 3; }) != 0;
    std::printf("%d %llu\n", found, (unsigned long long)(time - 1000));
  }
}
"""


def build(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def test_one_time_for_all_words_of_an_exchange(tmp_path):
    exe = build(tmp_path)

    def wait(ticks, *published):
        line = " ".join(map(str, (ticks, len(published)) + published))
        out = subprocess.run([exe], input=line, check=True, capture_output=True, text=True).stdout.split()
        return int(out[0]), int(out[1])

    assert wait(20000, *[0] * 8) == (8, 8)                    # all there: a look each
    found, took = wait(20000, *range(0, 16000, 2000))         # one after the other, within the time of the first
    assert found == 8 and 14000 <= took < 14100
    found, took = wait(20000, *[-1] * 8)                      # none: the time of one, not eight
    assert found == 0 and 20000 <= took < 20100
    found, took = wait(20000, 0, -1, 500, -1, 30000, 0, 19000, -1)   # what is there by then is still read
    assert found == 4 and 20000 <= took < 20100
    assert wait(0, 0, -1, 500, 0) == (2, 4)                   # no time: a look each


def test_time_from_a_text(tmp_path):
    """A decimal number up to 10 ms; anything else, numbers that would hold a workgroup for seconds among it, is the default."""
    texts = ["0", "1", "20000", "1000000", "1000001", "4294967295", "18446744073709551616", "-1", "", "soon", "10ms", " 5", "0x10"]
    out = subprocess.run([build(tmp_path)] + texts, check=True, capture_output=True, text=True).stdout.split()
    assert [int(x) for x in out] == [0, 1, 20000, 1000000] + [20000] * 10
