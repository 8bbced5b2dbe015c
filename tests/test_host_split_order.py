"""The order of the chained split Linears' tasks (split_order.h) run by threads on the host in place of workgroups: cleared
counters run every task once and after those it needs; counters that hold anything else, as when two calls overlap on one
workspace, still give tasks in range and an end."""
import subprocess

import pytest

SRC = r'''
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>
#include "split_order.h"
using namespace sm;
struct Mem {
  static int take(int* p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
  static int look(int* p) { return take(p, 0); }
  static int take_device(int* p, int v) { return take(p, v); }
  static void pause() { std::this_thread::yield(); }
};
int main(int argc, char** argv) {
  const int what = atoi(argv[1]), xcds = atoi(argv[2]), wgs = atoi(argv[3]), rows = atoi(argv[4]), groups = atoi(argv[5]);
  const int tiles_n[4] = {5, 8, 5, 3};
  int first[5] = {0};
  for (int i = 0; i < 4; ++i) first[i + 1] = first[i] + tiles_n[i] * rows;
  const int tasks = first[4], words = (4 * rows + SPLIT_LINE - 1) / SPLIT_LINE * SPLIT_LINE;
  std::vector<int> mem(SPLIT_LINE * 17 + groups * words, 0);
  std::vector<std::atomic<int>> ran((size_t)groups * tasks);
  for (auto& r : ran) r = 0;
  std::mt19937 rng(what);
  if (what) for (int& m : mem) m = what == 1 ? (int)rng() : what == 2 ? -1 : what == 3 ? 0x7fffffff : what == 4 ? (int)0x80000000 : (int)(rng() % 64);
  std::atomic<int> bad{0}, stop{0};
  auto workgroup = [&](int xcd) {
    int* mine = mem.data() + SPLIT_LINE * (1 + xcd);
    TaskOrder o{mem.data(), mine, (unsigned)tasks, groups, what ? 200u : 1u << 30, ~0u, 0, false};
    int to[2];
    task_of<Mem>(o, (unsigned)Mem::take(mine, 1), to);
    while (to[0] >= 0) {
      const int k = to[0], grp = to[1];
      if (k >= tasks || grp < 0 || grp >= groups) { ++bad; return; }
      int ph = 0;
      while (k >= first[ph + 1]) ++ph;
      int* done = mem.data() + SPLIT_LINE * 17 + grp * words + (k - first[ph]) % rows;
      if (ph) {
        wait_arrivals<Mem>(o, done + (ph - 1) * rows, tiles_n[ph - 1]);
        if (!what) for (int c = 0; c < tiles_n[ph - 1]; ++c)
          if (!ran[(size_t)grp * tasks + first[ph - 1] + c * rows + (k - first[ph]) % rows]) ++bad;
      }
      const unsigned n = (unsigned)Mem::take(mine, 1);
      ++ran[(size_t)grp * tasks + k];
      Mem::take(done + ph * rows, 1);
      task_of<Mem>(o, n, to);
    }
  };
  std::vector<std::thread> th;
  for (int x = 0; x < xcds; ++x) for (int w = 0; w < wgs; ++w) th.emplace_back(workgroup, x);
  std::thread clear([&] { if (what == 5) for (int i = 0; i < 50 && !stop; ++i) { for (int& m : mem) __atomic_store_n(&m, 0, __ATOMIC_SEQ_CST); std::this_thread::yield(); } });
  for (auto& t : th) t.join();
  stop = 1;
  clear.join();
  if (!what) for (auto& r : ran) if (r != 1) ++bad;
  printf("%d\n", (int)bad);
  return bad ? 1 : 0;
}
'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("split_order")
    (d / "t.cpp").write_text(SRC)
    import os
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_13528_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", csrc, str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


@pytest.mark.parametrize("xcds,wgs,rows,groups", [(8, 3, 1, 7), (8, 2, 10, 8), (3, 4, 2, 8), (1, 1, 3, 4), (8, 4, 1, 1)])
@pytest.mark.parametrize("what", range(6), ids=["cleared", "random", "ones", "largest", "lowest", "cleared while running"])
def test_tasks_in_order_or_an_end(program, what, xcds, wgs, rows, groups):
    for _ in range(3):
        r = subprocess.run([program] + [str(v) for v in (what, xcds, wgs, rows, groups)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
