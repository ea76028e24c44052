// Plans of the layers a thread has used lately (host side).  A plan depends on the operation, the descriptor, the room for
// partial sums and the tuning state only; making one (table search, then a cost model over every tile and split count) takes
// 0.4-8 us of host time, a look-up 0.05, a launch about 3, and a sequence of short layers was bound by it (ResNet-50 at batch
// 8, 64 x 64 images: 2.9 ms of host time per step against 2.1 ms of kernels).  One table per thread and precision that it
// launches convolutions in, fixed size (kPlanCacheSize entries, about 150 KB; kPlanCacheProbes of them looked at), so it
// cannot grow; a miss overwrites a stale entry among those or the first.
#pragma once
#include <string.h>

#include <memory>
#include <new>

#include "jz.h"

namespace jz {

struct PlanKey {
  int op, ca, cb;  // ca, cb: the residue of the stride the plan is for, -1 for a layer's own plan
  size_t limit;    // bytes of partial sums
  jz_conv_desc d;
};
constexpr unsigned kPlanCacheSize = 256, kPlanCacheProbes = 4;

template <class P>
struct PlanEntry {
  unsigned generation = 0;  // of the tuning state; 0: empty
  int rc = 0;
  PlanKey key{};
  P pl;
};
template <class P>
PlanEntry<P>* plan_table() {  // this thread's; nullptr: no memory for it
  thread_local std::unique_ptr<PlanEntry<P>[]> table(new (std::nothrow) PlanEntry<P>[kPlanCacheSize]);
  return table.get();
}

// *pl = the plan for the key, made by fill(pl) when it is not at hand; returns what fill returned for it.  generation: the
// tuning state's, never 0.  fill must not look plans of the same type up.
template <class P, class F>
int cached_plan(unsigned generation, const PlanKey& key, P* pl, F&& fill) {
  PlanEntry<P>* const table = plan_table<P>();
  if (!table) return fill(pl);
  const jz_conv_desc& d = key.d;
  const int words[15] = {key.op, key.ca, key.cb, (int)(key.limit >> 4), d.N, d.H, d.W, d.C, d.K, d.R, d.S, d.stride_h, d.stride_w, d.pad_h, d.pad_w};
  unsigned h = 2166136261u;
  for (int v : words) h = (h ^ (unsigned)v) * 16777619u;
  h ^= h >> 15;
  PlanEntry<P>* slot = &table[h % kPlanCacheSize];
  for (unsigned i = kPlanCacheProbes; i-- > 0;) {
    PlanEntry<P>& e = table[(h + i) % kPlanCacheSize];
    if (e.generation != generation) {
      slot = &e;
    } else if (e.key.op == key.op && e.key.ca == key.ca && e.key.cb == key.cb && e.key.limit == key.limit && memcmp(&e.key.d, &d, sizeof d) == 0) {
      *pl = e.pl;
      return e.rc;
    }
  }
  slot->generation = 0;
  slot->key = key;
  slot->pl = P{};
  slot->rc = fill(&slot->pl);
  slot->generation = generation;
  *pl = slot->pl;
  return slot->rc;
}

}  // namespace jz
