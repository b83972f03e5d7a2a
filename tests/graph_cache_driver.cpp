// The cache of captured steps (csrc/graph.hpp) on the host, over a stand-in for the HIP runtime.
#include <stdio.h>
#include <string.h>

#include <hip/hip_runtime.h>

#include "../paper_1710_07073_amd/csrc/graph.hpp"

namespace {

lbm::GraphKey key(int cur, int spar, bool marked) {
  return lbm::GraphKey::of(nullptr, nullptr, 3, cur, 0, 6, (uint32_t)(spar << 7) | (marked ? 4u : 0u));
}

template <class Cache>
void replay(Cache& c, const lbm::GraphKey& k, bool forked = false) {
  bool captured = false;
  c.ensure(k, nullptr, forked, [] { return hipSuccess; }, &captured);
  if (captured && forked)
    for (FakeGraph* g : fake.live)
      if (g->ended < g->launches) ++fake.captured_during;
  c.launch(nullptr);
}

// Calls of three replays of an odd number of pairs each: the buffers and the slab words flip with every replay,
// the first replay of a call has no box marked ahead. Prints the captures of the first two and of the later calls.
template <int N>
void flips() {
  fake = FakeHip{};
  {
    lbm::GraphCache<int, N> c;
    int parity = 0, first = 0;
    for (int call = 0; call < 12; ++call) {
      for (int i = 0; i < 3; ++i, parity ^= 1) replay(c, key(parity, parity, i > 0));
      if (call == 1) first = fake.captures;
    }
    printf("slots %d: captures %d, then %d, destroyed while running %d\n", N, first, fake.captures - first,
           fake.destroyed_running);
  }
  printf("  at the end: live %d, destroyed while running %d\n", (int)fake.live.size() - fake.destroyed,
         fake.destroyed_running);
}

// New keys faster than replays end, resets in between, and the cache gone during the last.
void storm(bool forked) {
  fake = FakeHip{};
  {
    lbm::GraphCache<int, 4> c;
    for (int i = 0; i < 200; ++i) {
      replay(c, key(i, 0, false), forked);
      if (i % 7 == 3) c.reset();
      if (i % 50 == 49)
        for (FakeGraph* g : fake.live) g->ended = g->launches;
    }
    printf("storm: captures %d, destroyed while running %d, waited %d, captured during replays %d\n", fake.captures,
           fake.destroyed_running, fake.waits > 0, fake.captured_during);
  }
  printf("  at the end: live %d, destroyed while running %d\n", (int)fake.live.size() - fake.destroyed,
         fake.destroyed_running);
}

}  // namespace

int main() {
  flips<4>();
  flips<2>();
  storm(false);
  storm(true);
  return 0;
}
