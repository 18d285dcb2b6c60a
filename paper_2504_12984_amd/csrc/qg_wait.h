// A wait for other wavefronts that has an end.
#pragma once

namespace qg {

// Under the rules of the interface what is waited for is already on its way, a few microseconds at most.  Calls that
// overlap on one workspace against the rules spoil each other's counters; their sums are wrong then, but
// the wait still ends: after LIMIT looks, of a microsecond each or less.
constexpr unsigned WAIT_LIMIT = 1u << 18;

// Whether count() came to `want` or beyond.
template <class Count, class Pause>
constexpr bool wait_for(Count count, unsigned want, Pause pause) {
  for (unsigned i = 0; i < WAIT_LIMIT; ++i) {
    if (count() >= want) return true;
    pause();
  }
  return false;
}

}  // namespace qg
