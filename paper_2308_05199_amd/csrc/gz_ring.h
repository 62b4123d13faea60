// gz_ring.h -- when an entry of the unit encoder's ring of rounds may be used
// again.  Plain integers, so that the rule that the kernels wait by is the one
// that a host model runs (tests/ring_model.cpp).
#pragma once
#include <stdint.h>

namespace gzk {

constexpr uint32_t RING = 8;

// Round k of a workgroup sits in entry k % RING, with a count of the sizes its
// workers have published and a mark (1 + round) that the scheduler sets once
// it needs nothing more of the entry but its aggregate's mark.
// Before round k is opened:
//   * the workers have published round k - 2: they wait for no earlier ticket,
//     and hold no unit older than round k - 4 (round k - RING's entry, which
//     round k takes, is read by none of them);
//   * the scheduler is done with round k - RING.  The workers alone do not say
//     so: one whose units were dropped (a malformed incoming superblock, an
//     expired wait) waits for no prefix and may be any number of rounds ahead.
struct RingNeed {
  bool published, scheduled;  // whether there is such a round
  uint32_t pub;               // entry whose count has to reach the workers' number
  uint32_t sched, mark;       // entry whose mark has to reach `mark`
};

constexpr RingNeed ring_need(uint32_t k) {
  return RingNeed{k >= 2, k >= RING, (k - 2) % RING, k % RING, k - RING + 1};
}

}  // namespace gzk
