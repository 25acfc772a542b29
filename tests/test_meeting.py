"""The meeting of the workgroups that share a result (csrc/exchange.h), its source run by threads of the CPU: every share is finished once,
behind the last arrival, whether its member waits, leaves at once or leaves late, launch after launch in the same word."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_00264_amd", "csrc")

MAIN = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#define __device__ static
#define __forceinline__ inline
#include "exchange.h"
struct Word {
  std::atomic<unsigned>* p;
  unsigned add(unsigned v) const { return p->fetch_add(v); }
  unsigned load() const { if (rand() % 3 == 0) std::this_thread::yield(); return p->load(); }
  void store(unsigned v) const { p->store(v); }
  bool swap(unsigned from, unsigned to) const { return p->compare_exchange_strong(from, to); }
};
int main() {
  std::atomic<unsigned> word{0};
  long left = 0;
  for (int round = 0; round < 3000; ++round) {               // (the count of finished meetings wraps at 256)
    const unsigned S = 1 + round % 16;
    const int polls = round % 4 == 0 ? 0 : round % 4 == 1 ? 1 : round % 4 == 2 ? 3 : 1 << 30;
    std::atomic<unsigned> here{0}, start{0};
    std::vector<std::atomic<int>> done(S);
    std::atomic<int> bad{0}, gone{0};
    std::vector<std::thread> t;
    for (unsigned i = 0; i < S; ++i)
      t.emplace_back([&, i] {
        ++start;
        while (start < S) std::this_thread::yield();
        for (int k = rand() % 200; k > 0; --k) word.load();
        ++here;
        const unsigned todo = meet(Word{&word}, S, i, polls);
        if (todo != 0 && here != S) ++bad;
        if (todo >> S) ++bad;
        if (todo == 0) ++gone;
        for (unsigned j = 0; j < S; ++j) if (todo >> j & 1) ++done[j];
      });
    for (auto& x : t) x.join();
    for (auto& d : done) if (d != 1) ++bad;
    if (polls == 1 << 30 && gone != 0) ++bad;
    if ((word & 0xffffff) != 0 || word >> 24 != ((unsigned)round + 1) % 256) ++bad;
    left += gone;
    if (bad) { printf("round %d, %u members, %d polls\n", round, S, polls); return 1; }
  }
  return left > 0 ? 0 : 2;                                   // (some did leave)
}
"""


def test_every_share_is_finished_once(tmp_path):
    (tmp_path / "k.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(tmp_path / "k.cpp"), "-o", str(tmp_path / "k")], check=True)
    r = subprocess.run([str(tmp_path / "k")], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.returncode, r.stdout)
