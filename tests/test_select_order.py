"""The order in which a selection launch's workgroups take their camera groups
(csrc/group_order.h), built for the CPU: workgroups that start in any order, with
fewer places than workgroups, must all end, whichever wait for the one before. The
same program with the workgroup's number in place of the ticket shows that the
orders it tries are ones in which a wait would never end (its waits are bounded)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_30459_amd", "csrc")

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "group_order.h"

static std::atomic<long> pauses{0};
static const long kPauses = 20000;  // looks at an entry after which a wait counts as endless
struct Stuck {};
struct HostMem {
  template <class T> static T add(T* p, T v) { return __atomic_fetch_add(p, v, __ATOMIC_RELAXED); }
  template <class T> static T load(T* p) { return __atomic_load_n(p, __ATOMIC_RELAXED); }
  template <class T> static void store(T* p, T v) { __atomic_store_n(p, v, __ATOMIC_RELAXED); }
  static void pause() {
    if (++pauses > kPauses) throw Stuck();
    std::this_thread::yield();
  }
};

// argv: use tickets, groups, groups a stream, places, seed of the start order (0: last first), launches
int main(int, char** a) {
  const bool tickets = atoi(a[1]);
  const int n = atoi(a[2]), per = atoi(a[3]), places = atoi(a[4]), launches = atoi(a[6]);
  unsigned seed = atoi(a[5]);
  std::vector<int64_t> chain(n, 0), next_id(n, 100);
  int32_t ticket = 0;
  for (int launch = 0; launch < launches; ++launch) {
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = n - 1 - i;
    if (seed)
      for (int i = n - 1; i > 0; --i) {
        seed = seed * 1664525u + 1013904223u;
        std::swap(order[i], order[(seed >> 8) % (i + 1)]);
      }
    std::vector<int64_t> got(n, -1);
    std::atomic<int> started{0};
    std::atomic<bool> stuck{false};
    pauses = 0;
    // a place starts the next workgroup of the order when its last one has ended
    auto place = [&] {
      for (int i; (i = started++) < n;) {
        try {
          const int g = tickets ? vio::take_group<HostMem>(&ticket, n) : order[i];
          const int s = g / per;
          const bool first = g % per == 0, last = g % per == per - 1 || g == n - 1;
          const int64_t id = first ? next_id[s] : vio::take_id<HostMem>(&chain[g - 1]);
          got[g] = id;
          if (last) next_id[s] = id + g;
          else vio::hand_on_id<HostMem>(&chain[g], id + g);
        } catch (const Stuck&) {
          stuck = true;
          return;
        }
      }
    };
    std::vector<std::thread> t;
    for (int p = 0; p < places; ++p) t.emplace_back(place);
    for (auto& x : t) x.join();
    if (stuck) return puts("stuck"), 0;
    int64_t want = 0;
    static std::vector<int64_t> base(n, 100);
    for (int g = 0; g < n; ++g) {
      if (g % per == 0) want = base[g / per];
      if (got[g] != want) return puts("wrong"), 0;
      want += g;
      if (g % per == per - 1 || g == n - 1) base[g / per] = want;
    }
    if (ticket != 0) return puts("ticket"), 0;
    for (int64_t c : chain)
      if (c != 0) return puts("chain"), 0;
  }
  puts("ok");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(PROGRAM)
    exe = str(d / "order")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(d / "order.cpp"), "-o", exe], check=True)
    return lambda *a: subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True,
                                     timeout=60).stdout.strip()


@pytest.mark.parametrize("groups,per,places", [(2, 2, 1), (3, 3, 2), (64, 2, 1), (64, 2, 8), (64, 64, 5), (17, 4, 3),
                                               (64, 1, 3)])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_every_wait_ends(program, groups, per, places, seed):
    assert program(1, groups, per, places, seed, 5) == "ok"


def test_the_order_of_numbers_would_not(program):
    assert program(0, 2, 2, 1, 0, 1) == "stuck"
    assert program(0, 64, 64, 5, 0, 1) == "stuck"
