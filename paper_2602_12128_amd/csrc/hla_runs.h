// How a call's tokens are cut into runs on the generic path (host only; no HIP in this file).
#ifndef HLA_RUNS_H_
#define HLA_RUNS_H_

#include <algorithm>
#include <cstdint>

namespace hla {

// Tiles per run: the fewest, from the share of one of `cap` runs on, with which the runs of all heads
// stay within `cap` or every sequence is one run.  count(per): runs of one head with `per` tiles each;
// it costs a pass over the sequences and never grows with `per`, so the search doubles and then halves
// its step.  Host time of a forward with one sequence of 32760 tokens and the rest of 20, 12 heads: 64
// sequences 30 us, 2000 sequences 89 us; counting tile by tile, in every call, 112 and 2277 us.
template <class Count>
inline int64_t tiles_per_run(int64_t heads, int64_t nseq, int64_t cap, Count&& count) {
  auto fits = [&](int64_t per) {
    const int64_t c = count(per);
    return c * heads <= cap || c <= nseq;
  };
  int64_t lo = std::max<int64_t>(1, count(1) * heads / cap);
  if (fits(lo)) return lo;
  int64_t step = 1;
  while (!fits(lo + step)) {
    lo += step;
    step *= 2;
  }
  int64_t hi = lo + step;  // fits; lo does not
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    (fits(mid) ? hi : lo) = mid;
  }
  return hi;
}

}  // namespace hla

#endif  // HLA_RUNS_H_
