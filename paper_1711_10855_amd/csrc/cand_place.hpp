// Places in the list of candidates that a block of a detection kernel keeps in
// LDS (see CandLds). Plain C++: the counting also runs on the host.
#pragma once

namespace fdas {

constexpr int kCandLds = 320;

// Where an offer of `total` candidates goes: its first entry, to be tested with
// cand_fits. `taken` reads how many entries were asked for so far, `take` adds
// to them and returns what they were. Once the list is full nothing is added:
// a unit may hold every row of its segments, whose hits pass 2^31 (131089 rows
// of 16384 points at threshold 0), and a count that wraps would fit again. Each
// wave may still add the one offer for which it read a list that was not full.
template <class Taken, class Take>
constexpr int cand_place(int total, Taken taken, Take take) {
  return taken() < kCandLds ? take(total) : kCandLds;
}

constexpr bool cand_fits(int pos, int total) { return pos + total <= kCandLds; }

// Entries of a finished list: `lim` is the least place of an offer that did not
// fit (kCandLds without one).
constexpr int cand_listed(int n, int lim) { return n < lim ? n : lim; }

}  // namespace fdas
