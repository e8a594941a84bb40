// The autotuner's walk over kernel variants, apart from how a variant is run:
// host code without device calls.
#pragma once

namespace mpmx {

struct TuneChoice {
  int p2g, g2p, g2p_adj, p2g_adj, box, specialize, fuse, fuse_adj, xcd, grid_list;
};

// the plain mode's kernels: what every other choice is compared with
constexpr TuneChoice kTuneReference{0, 0, 0, 0, 0, 1, 0, 0, 0, 0};

// Finds the fastest choice that agrees with the reference. attempt(choice, bwd,
// ms, agrees) runs a choice, times it (forward only or with the backward) and
// compares its end state and its cotangents with the reference's; it returns 0,
// or an error that ends the walk. over_budget() stops further candidates. `best`
// is a choice that agreed, or the reference itself, at every step and on return.
template <typename Attempt, typename OverBudget>
int tune_choice(Attempt&& attempt, OverBudget&& over_budget, TuneChoice& best) {
  best = kTuneReference;
  // the first of these that agrees is where one option after another is tried from: the defaults, then the same
  // without the fused kernels (a fault in one of those would otherwise hide the unfused ones)
  constexpr TuneChoice starts[] = {{2, 1, 2, 1, 0, 1, 1, 1, 0, 0}, {2, 1, 2, 1, 0, 1, 0, 0, 0, 0}};
  for (const TuneChoice& c : starts) {
    double ms = 0.0;
    bool agrees = false;
    const int rc = attempt(c, true, ms, agrees);
    if (rc) return rc;
    if (agrees) { best = c; break; }
  }
  struct Group {
    int TuneChoice::*option;
    int n, values[3];
    bool bwd;   // timed with the backward
  };
  constexpr Group groups[] = {
      {&TuneChoice::p2g, 2, {2, 0}, false},        {&TuneChoice::g2p_adj, 2, {2, 0}, true},
      {&TuneChoice::box, 2, {0, 1}, true},         {&TuneChoice::specialize, 2, {1, 0}, true},
      {&TuneChoice::fuse, 2, {1, 0}, true},        {&TuneChoice::fuse_adj, 2, {1, 0}, true},
      {&TuneChoice::xcd, 2, {0, 1}, true},         {&TuneChoice::grid_list, 3, {0, 1, 2}, true},
  };
  for (const Group& grp : groups) {
    const TuneChoice keep = best;
    double best_ms = 1e30;
    for (int i = 0; i < grp.n; ++i) {
      if (over_budget()) return 0;
      TuneChoice trial = keep;
      trial.*grp.option = grp.values[i];
      double ms = 0.0;
      bool agrees = false;
      const int rc = attempt(trial, grp.bwd, ms, agrees);
      if (rc) return rc;
      // a later candidate must win by more than 1%: a tie keeps the earlier (default) choice, so timing noise does
      // not flip between equivalent variants
      if (agrees && ms < best_ms * 0.99) {
        best_ms = ms;
        best = trial;
      }
    }
  }
  return 0;
}

}  // namespace mpmx
