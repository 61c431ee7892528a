// Counting the loads of the GEMM's LDS ring; plain C++, so that the host can
// check it too.
#pragma once

namespace lmop {

// A wave's loads land in the order of their issue, so a stage has landed once
// no more loads are in flight than were issued after it.  Every stage is
// `loads` loads, and the last `pf` of the kt_n stages carry one more (the
// residual prefetch).  Of the `fly` stages that end with stage `newest`,
// these are in flight at most; where only the newer ones carry the further
// load, the count leaves it out (a smaller count only waits for more).
constexpr bool all_carry_prefetch(int newest, int fly, int kt_n, int pf) {
  return newest - fly + 1 >= kt_n - pf;
}

}  // namespace lmop
