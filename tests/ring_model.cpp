// Host model of one workgroup of the unit encoder: `W` workers and the scheduler
// take steps in random order over the ring of round entries, and an entry is
// used again by the kernels' own rule (gz_ring.h).  Units are dropped (never held:
// malformed, so that their worker waits for no prefix) with probability `drop`
// percent, and the scheduler takes a step with weight 1 against `lag`.
// Prints "ok", or what went wrong: the scheduler or a worker used an entry of
// another round, or nobody could take a step.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gz_ring.h"
using namespace gzk;

struct Entry {
  uint32_t ticket = 0, ready = 0, cnt = 0, pready = 0, sum = 0, size[16] = {};
};
static uint32_t size_of(uint32_t ticket, uint32_t w) { return 1 + ticket * 16 + w; }

struct Worker {
  uint32_t k = 0, step = 0, tk = 0;
  bool first = false, done = false;
  std::vector<uint32_t> held;  // rounds of its held units, the oldest first
};

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const uint32_t W = atoi(argv[1]), total = atoi(argv[2]), drop = atoi(argv[3]), lag = atoi(argv[4]);
  std::mt19937 g(atoi(argv[5]));
  std::vector<Entry> rs(RING);
  std::vector<Worker> ws(W);
  uint32_t next = 0;
  uint32_t sk = 0, sstep = 0, st = 0;  // scheduler: round, step, ticket read
  bool sdone = false;
  auto open = [&](uint32_t k, uint32_t t) {
    Entry& e = rs[k % RING];
    e.cnt = 0;
    e.ticket = t;
    e.ready = k + 1;
  };
  open(0, next++);
  auto fail = [&](const char* s, uint32_t k) { printf("%s at round %u\n", s, k); exit(1); };

  auto sched = [&]() -> bool {
    Entry& e = rs[sk % RING];
    if (sstep == 0) {
      if (e.ready < sk + 1) return false;
      st = e.ticket;
      if (st != sk) fail("the scheduler read another round's ticket", sk);
      if (st >= total) sdone = true;
      else sstep = 1;
    } else if (sstep == 1) {
      if (e.cnt < W) return false;
      e.sum = 0;
      for (uint32_t w = 0; w < W; ++w) {
        if (e.size[w] != size_of(st, w)) fail("the scheduler read another round's sizes", sk);
        e.sum += e.size[w];
      }
      sstep = 2;
    } else {  // after the look-back
      if (e.ready != sk + 1) fail("the entry was opened again under the scheduler", sk);
      e.pready = sk + 1;
      ++sk;
      sstep = 0;
    }
    return true;
  };
  // a worker's oldest held unit: its prefix must be its round's
  auto flush = [&](Worker& x, uint32_t w) -> bool {
    const uint32_t k = x.held.front();
    Entry& e = rs[k % RING];
    if (e.pready < k + 1) return false;
    if (e.pready != k + 1 || e.ticket != k || e.size[w] != size_of(k, w))
      fail("a worker wrote a unit by another round's entry", k);
    x.held.erase(x.held.begin());
    return true;
  };
  auto work = [&](uint32_t w) -> bool {
    Worker& x = ws[w];
    Entry& e = rs[x.k % RING];
    switch (x.step) {
      case 0:  // the round's ticket
        if (e.ready < x.k + 1) return false;
        if (e.ready != x.k + 1) fail("a worker read another round's ticket", x.k);
        if (e.ticket >= total) {
          if (x.held.empty()) x.done = true;
          else return flush(x, w);
          return true;
        }
        x.step = 1;
        return true;
      case 1:  // publish
        e.size[w] = size_of(e.ticket, w);
        x.first = ++e.cnt == 1;
        x.step = 2;
        return true;
      case 2:  // write what is two rounds old
        if (!x.held.empty() && x.held.front() + 1 < x.k) return flush(x, w);
        if (x.first) x.tk = next++;
        x.step = 3;
        return true;
      default: {  // open the next round, hold the unit or drop it
        if (x.first) {
          const RingNeed n = ring_need(x.k + 1);
          if (n.published && rs[n.pub].cnt < W) return false;
          if (n.scheduled && rs[n.sched].pready < n.mark) return false;
          open(x.k + 1, x.tk);
        }
        if (g() % 100 >= drop) x.held.push_back(x.k);
        ++x.k;
        x.step = 0;
        return true;
      }
    }
  };
  for (;;) {
    bool all = sdone;
    for (auto& x : ws) all = all && x.done;
    if (all) break;
    // one actor's step; if none of a long run can move, all are asked once
    bool moved = false;
    for (uint32_t i = 0; i < 4 * (W + 1) && !moved; ++i) {
      const uint32_t a = g() % (W * lag + 1);
      moved = a == W * lag ? (!sdone && sched()) : (!ws[a % W].done && work(a % W));
    }
    if (!moved) {
      if (!sdone) moved = sched();
      for (uint32_t w = 0; w < W; ++w) moved = (!ws[w].done && work(w)) || moved;
      if (!moved) fail("nobody can take a step", sk);
    }
  }
  puts("ok");
  return 0;
}
