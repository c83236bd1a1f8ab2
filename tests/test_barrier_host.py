"""The host side of the grid barrier (la_barrier.h, plain C++): small programs run it, without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_16760_amd", "csrc")

EPOCHS = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "la_barrier.h"
using namespace la;
// The barrier words as one number: the largest epoch that a launch has left (counters: arrivals per member).
int main(int, char **v) {
  const bool counters = atoi(v[1]) != 0;
  const unsigned layers = (unsigned)atoi(v[2]);
  std::mt19937 rng((unsigned)atoi(v[3]));
  BarrierEpochs e;
  e.init(5 * layers > 2 ? 5 * layers : 2, counters);
  struct Node { unsigned epoch0, n; bool clear; };
  std::vector<Node> graph;
  unsigned words = 0, restarts = 0, wrong = 0, highest = 0;
  auto run = [&](const Node &k) {
    if (k.clear) words = 0;
    if (counters ? words != k.epoch0 : words > k.epoch0) ++wrong;
    words = k.epoch0 + k.n;
    if (words > highest) highest = words;
  };
  for (int i = 0; i < atoi(v[4]); ++i) {
    const unsigned n = rng() % 2 ? 2 : 5 * (1 + rng() % layers), what = rng() % 1000000 == 0 ? 100 : rng() % 100;
    if (what == 0) {  // a graph of one to three launches; nothing runs yet
      graph.clear();
      for (unsigned k = rng() % 3 + 1; k > 0; --k) {
        const auto l = e.launch(n, true);
        graph.push_back({l.epoch0, n, l.clear});
      }
    } else if (what < 30) {
      for (const auto &k : graph) run(k);
    } else if (what == 100) {  // recovery after an error, in a graph that is never run or on a stream
      const bool capturing = rng() % 2;
      e.cleared(capturing);
      if (!capturing) words = 0;
    } else {
      const auto l = e.launch(n, false);
      restarts += l.clear;
      run({l.epoch0, n, l.clear});
    }
  }
  printf("%u %u %u\n", wrong, restarts, highest);
}
"""

PATIENCE = r"""
#include <cstdio>
#include <cstdlib>
#include "la_barrier.h"
using namespace la;
int main(int, char **v) {
  const unsigned units = barrier_patience((unsigned)strtoul(v[1], nullptr, 10));
  // the first poll that ends the wait, by bisection over what a 32-bit count of polls can say; 0: none
  unsigned long long lo = 0, hi = 1ull << 32;
  while (lo + 1 < hi) {
    const unsigned long long mid = (lo + hi) / 2;
    (patience_over((unsigned)mid, units) ? hi : lo) = mid;
  }
  printf("%u %llu\n", units, hi < 1ull << 32 ? hi : 0);
}
"""

DEAD = r"""
#include <cstdio>
#include <cstdlib>
#include "la_barrier.h"
int main(int, char **v) {
  const unsigned units = (unsigned)atoi(v[1]), dies = (unsigned)atoi(v[2]);  // another wave marks the workgroup before this poll
  unsigned polls = 0, looks = 0;
  while (!la::wait_over(polls, units, [&]() { ++looks; return polls >= dies; })) {}
  printf("%u %u\n", polls, looks);
}
"""


def _program(tmp_path_factory, name, text):
    d = tmp_path_factory.mktemp(name)
    (d / "main.cpp").write_text(text)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)
    return lambda *a: [int(x) for x in subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout.split()]


@pytest.fixture(scope="module")
def epochs(tmp_path_factory):
    return _program(tmp_path_factory, "epochs", EPOCHS)


@pytest.mark.parametrize("layers", [1, 2, 40])
@pytest.mark.parametrize("counters", [0, 1])
def test_no_launch_finds_words_that_have_reached_its_epochs(epochs, counters, layers):
    """Launches, graphs of launches and their replays in any order.  40 layers: the epochs restart (past 2^26)."""
    wrong, restarts, highest = epochs(counters, layers, 7, 4_000_000)
    assert wrong == 0 and highest < 1 << 30
    if layers == 40 and not counters:
        assert restarts >= 1


@pytest.fixture(scope="module")
def patience(tmp_path_factory):
    return _program(tmp_path_factory, "patience", PATIENCE)


@pytest.mark.parametrize("asked,units", [(0, 1 << 21), (1, 1), (1000, 1000), ((1 << 30) - 2, (1 << 30) - 2), ((1 << 30) - 1, (1 << 30) - 2),
                                         (1 << 30, (1 << 30) - 2), ((1 << 32) - 1, (1 << 30) - 2)])
def test_every_wait_ends(patience, asked, units):
    """Whatever la_set_barrier_timeout was given: a wait's 32-bit count of polls reaches its end, four polls a unit."""
    assert patience(asked) == [units, 4 * (units + 1)]


@pytest.mark.parametrize("units,dies,polls", [(1 << 21, 1, 256), (1 << 21, 256, 256), (1 << 21, 257, 512), (1 << 21, 5_000_000, 5_000_192), (1, 1, 8),
                                              (1000, 1 << 30, 4004)])
def test_a_wait_ends_with_its_workgroup(tmp_path_factory, units, dies, polls):
    """At the next look at the mark, long before its own patience; a look is every 256 polls."""
    assert _program(tmp_path_factory, "dead", DEAD)(units, dies) == [polls, polls // 256]
