// The slabs of a unit, nk >= 2 of them, in which a scheduling wave takes the steps that end in the description of the unit after the
// next: it claims a unit, asks for the plan's entry, for the rows of the token map and for the completion counter of the unit's chunk, and
// publishes.  Each step uses what the one before it brought, so a step may share a slab with the one before (the kernels run them in this
// order inside a slab) but never come ahead of it: a counter that is read for the unit claimed before would mark rows as stored that are not.
// Plain C++ and no other header, so that the order can also be checked on the host (tests/test_ffn_steps_cpu.py).
#pragma once

namespace ew {

struct SchedSteps {
  int claim, entry, rows, stored, publish;
};

// k_ffn_dec: spread over the whole unit, the claim in its first slab.
constexpr SchedSteps steps_spread(int nk) {
  const int n = nk - 2;
  return {0, n / 3, 2 * n / 3, n > 0 ? n - 1 : 0, n};
}

// k_ffn_big: as late as kStepGap slabs (2.5 to 3 us) from claim to entry to rows to publication allow; contractions of fewer than eight slabs
// have one slab in between, those of two to four none.  The counter last, one slab ahead where there is one.
constexpr int kStepGap = 2;
constexpr SchedSteps steps_late(int nk) {
  const int n = nk - 2, gap = n / 3 < kStepGap ? n / 3 : kStepGap;
  return {n - 3 * gap, n - 2 * gap, n - gap, n - (gap < 1 ? gap : 1), n};
}

// Published before the unit's last slab, behind whose barrier the description is read.
constexpr bool steps_in_order(const SchedSteps& s, int nk) {
  return 0 <= s.claim && s.claim <= s.entry && s.entry <= s.rows && s.rows <= s.stored && s.stored <= s.publish && s.publish == nk - 2;
}
// (From eight slabs on three more of them move every step of the one by 0, 1, 2, 3 and 3 slabs and all of the other by three.)
constexpr bool steps_in_order_up_to(int most) {
  for (int nk = 2; nk <= most; ++nk)
    if (!steps_in_order(steps_spread(nk), nk) || !steps_in_order(steps_late(nk), nk)) return false;
  return true;
}
static_assert(steps_in_order_up_to(256), "a scheduling step ahead of the one whose result it uses");

}  // namespace ew
