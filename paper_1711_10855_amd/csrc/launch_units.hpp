// How launches are cut into work units: of a single spectrum, and the items of a
// batch. Plain C++: the choices also run on the host.
#pragma once

#include <algorithm>
#include <cstdint>
#include <utility>

namespace fdas {

// What the time of a launch depends on, in templates of one row in full company
// (every slot of the GPU's blocks taken): see UnitCost.
struct UnitModel {
  double forward;  // a unit's forward transform
  double alone;    // a block's time alone, as a share of that in full company
  double fixed;    // the share that does not shrink with fewer blocks around it
  double step;     // how far blocks keep step (1: in rounds, 0: as slots fall free)
  double single;   // a row of the single form against one of the pair form
  // What a template takes longer in a unit of 100 rows or more (and in proportion
  // in a shorter one) on ragged planes, in the pair and in the single form.
  double ragged[2];
};

// Units of a launch: every row of the first n1 segment groups, then zpb2 rows at
// a time of the others (zpb1 rows where n1 is given; see UnitGrid).
struct UnitSplit {
  int64_t n1;
  int zpb1, zpb2;
  int pair;  // rows z and -z together
};

// Estimated time of a launch over nsb segment groups, n1 of them in whole-row
// units that fill k rounds of the `slots` block slots, the others in groups of
// `per` of the n rows (or pairs of rows) each.
//
// Two limits bound it. Blocks that start together and are alike end together,
// so that a launch runs in rounds as long as a unit; a last round with fewer
// blocks ends sooner, as a block shares its SIMDs with fewer others, down to
// `alone` of its time (by whole blocks on a compute unit). Blocks that drift
// apart fill the slots as they fall free: the time is that of all the work
// spread over the slots, and a share of one unit for the end. Which one it is
// differs by kernel: blocks of one wave share a SIMD four ways and drift, a
// block of 16 waves holds half a compute unit and keeps step.
//
// A plane that the caches do not hold, whose rows or segments do not lie on 64
// bytes, is ragged: where two segments or two stores of one meet in a line, the
// line is written twice unless both halves come soon after one another, which
// they do the less the more rows a unit has. (2048 points, m = 250, 2^22 bins x
// 101 rows: units of 102 rows 758 us, 52 695, 34 671, 18 629; m = 256, aligned: 576,
// 558, 553, 584.)
//
// The constants are fitted to measured times of 5 numbers of rows (17 .. 201) x
// 14 lengths (15000 .. 2^23 bins) in up to 50 layouts each; what the estimate
// picks takes on average 1.01 times the fastest of them at 256 to 1024 points,
// 1.005 times at the others. (256 points, 202 rows of single form, 1366 groups
// on 4096 slots: units of 202 rows 203 us, 101 150, 41 140, 21 137, 9 155. 2048
// points, 101 rows, 140 segments on 1024 slots: units of 102 rows 162 us, 22
// 46.8, 16 43.0, 14 44.0, 12 52.7, 2 82.6. Units counted in whole rounds alone,
// with one size for the end of a launch, took 1.33 times as long at worst: 102
// rows x 1100000 bins at 256 points 187 us, where units of 34 rows take 141.)
struct UnitCost {
  UnitModel m;
  int64_t nsb, slots;
  int cus, nz, each;  // each: rows counted by one of n
  double ragged;      // of UnitModel's for this form, or 0

  double operator()(int64_t k, int per) const {
    const int n = (nz + each - 1) / each, groups = (n + per - 1) / per;
    const double rest = (double)(nsb - k * slots), units = rest * groups;
    const double full = (double)(int64_t)(units / (double)slots);
    const double left = units - full * (double)slots;
    const int rows = std::min(each * per, nz);
    const double longer = 1.0 + ragged * std::min(rows, 100) * 0.01;
    const double all = (nz + m.forward) * (1.0 + ragged * std::min(nz, 100) * 0.01);
    const double unit = rest == 0.0 ? all : (rows + m.forward) * longer;
    const double work =
        rest / (double)slots * (nz + m.forward * groups) * longer + (double)k * all;
    const double spread = std::max(m.alone * unit, m.fixed * unit + (1.0 - m.fixed) * work);
    double last = 0.0;
    if (left > 0.0) {
      const double share = (double)(int64_t)((left + cus - 1) / cus) * cus / (double)slots;
      last = std::max(m.alone, m.fixed + (1.0 - m.fixed) * share);
    }
    const double rounds = (double)k * all + (full + last) * unit;
    return (double)slots * (m.step * rounds + (1.0 - m.step) * spread);
  }

  // No layout of k whole-row rounds and `groups` or more groups costs less.
  double least(int64_t k, int groups) const {
    const double work = (double)(nsb - k * slots) * (nz + m.forward * groups) +
                        (double)(k * slots) * (nz + m.forward);
    return (1.0 - m.fixed * (1.0 - m.step)) * work;
  }
};

// The cheapest of: no whole-row units, or as many rounds of them as the groups
// fill, or one less, and the rest in any number of near-equal row groups; in the
// pair form (pair_slots > 0) or, without whole-row units, in the single form,
// whose units may have an odd number of rows. Only layouts that can be the
// cheapest are looked at: of those whose blocks all run alone the finest, and
// then finer ones until the forward transforms alone cost more. `looked`, if
// given, counts them.
inline UnitSplit pick_units(const UnitModel &m, int64_t nsb, int nz, int cus, int64_t pair_slots,
                            int64_t single_slots, bool ragged, int64_t *looked = nullptr) {
  UnitSplit best{0, nz, nz, pair_slots > 0};
  double best_cost = -1.0;
  const double few = m.fixed < 1.0 ? std::max(0.0, (m.alone - m.fixed) / (1.0 - m.fixed)) : 0.0;
  for (int pair = pair_slots > 0 ? 1 : 0; pair >= 0; --pair) {
    const int64_t slots = pair ? pair_slots : single_slots;
    if (slots <= 0) continue;
    const double factor = pair_slots > 0 && !pair ? m.single : 1.0;
    const UnitCost cost{m, nsb, slots, cus, nz, pair ? 2 : 1, ragged ? m.ragged[pair ? 0 : 1] : 0.0};
    const int n = (nz + cost.each - 1) / cost.each;
    // (the single form of a plan with pairs: without whole-row units only)
    const int64_t full = pair || pair_slots <= 0 ? nsb / slots : 0;
    for (int64_t k = full;; k = k == full && full > 1 ? full - 1 : 0) {
      const int64_t rest = nsb - k * slots;
      int64_t g = 1;
      if (k == 0 && rest > 0)
        g = std::max<int64_t>(1, (int64_t)(few * (double)slots / cus) * cus / rest);
      g = std::min<int64_t>(g, n);
      for (int per = (int)((n + g - 1) / g);;) {
        const int groups = (n + per - 1) / per;
        if (best_cost >= 0.0 && factor * cost.least(k, groups) >= best_cost) break;
        const double c = factor * cost(k, per);
        if (looked) ++*looked;
        if (best_cost < 0.0 || c < best_cost * 0.999) {
          best_cost = c;
          best = {k * slots, nz, std::min(cost.each * per, nz), pair};
        }
        if (per == 1 || rest == 0) break;
        const int next = (n + per - 2) / (per - 1);  // fewest groups of less than per
        per = (n + next - 1) / next;
      }
      if (k == 0) break;
    }
  }
  return best;
}

// What the time of a batch depends on, in templates of one row: what an item
// takes beside its rows (its forward transform, and the wait for the next item,
// which counts most where a block is one wave), the share of an item for the
// uneven end, and a block's time alone as a share of that in full company.
struct BatchModel {
  double item, end, alone;
  // As in UnitModel, for planes ragged in their rows and in their segments.
  double ragged_rows, ragged_segments;
};

// Work items of a batch, its series in the order in which blocks take them
// (largest first): one item per (series, segment group) with all rows, which pays
// the forward transform once, but for the series from `tail` on, which make up
// the last round of the GPU's block slots: those in near-equal groups of at most
// `zpb` rows, so that the blocks end together. The size is the one whose work,
// spread over the slots, and the share of an item for the end are least; a batch
// of less than a round is all tail, and its blocks run in rounds as those of a
// single spectrum do. The constants of the FP32 kernels are fitted to 16 batches in
// up to 60 layouts each; what this picks takes on average 1.01 times the fastest
// of them at 256, 512 and 4096 points, 1.02 at 2048, 1.03 at 1024 and in 16
// bits. (5 series of 20
// segments and 201 rows in FP32 on 512 slots: items of 34 rows, 0.82 rounds, 110
// us; of 26, 1.09, 137; of 14, 2.05, 112. 12 series of 2^19 .. 2^21 bins and 33
// .. 101 rows in FP32: 1302 us in groups of at most 40 rows, 1257 this way; 6
// series of 95000 .. 190000 bins in FP16: 116 against 86 us. With one price of 3
// rows for every FP32 item, 3 series of 220 segments and 26 rows at 512 points
// went in items of 4: 50 us, 30 in items of 14.)
struct BatchUnits {
  int tail, zpb;
};

// Ragged planes (`ragged`: the model's, else 0) are all tail: their items are short
// for the same reason as the units above. (4 series of 2^20 bins x 101 rows at 2048
// points, m = 250: 655 us whole, 634 this way. At 512 points 2 series of 3000001
// bins and odd rows: 802, 745. Odd rows at 2048 points with m = 256 are no slower
// whole.)
//
// get(k): segment groups and rows of the series at place k of n. The tail is
// summed by its numbers of rows, of which there are few (beyond kKinds the
// others count as the last), so that the many sizes tried cost little however
// many series there are: 2000 one-segment series took 60 us of host time.
template <class Get>
inline BatchUnits pick_batch(const BatchModel &m, int64_t slots, int cus, bool pair, double ragged,
                             int n, Get &&get) {
  constexpr int kKinds = 64;
  int rows = 0;
  for (int k = 0; k < n; ++k) rows = std::max(rows, get(k).second);
  struct {
    int rows;
    int64_t groups;
  } kind[kKinds];
  int kinds = 0, tail = n, tail_rows = 1;
  double work = 0.0, head = 0.0;
  while (tail > 0 && (ragged > 0.0 || work < (double)slots * (rows + m.item))) {
    const std::pair<int64_t, int> x = get(--tail);
    work += (double)x.first * (x.second + m.item);
    tail_rows = std::max(tail_rows, x.second);
    int i = 0;
    while (i < kinds && kind[i].rows != x.second) ++i;
    if (i == kKinds) i = kKinds - 1;
    if (i == kinds) kind[kinds++] = {x.second, 0};
    kind[i].groups += x.first;
  }
  for (int k = 0; k < tail; ++k) {
    const std::pair<int64_t, int> x = get(k);
    head += (double)x.first * (x.second + m.item);
  }
  BatchUnits best{tail, tail_rows};
  double best_time = -1.0;
  for (int groups : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32}) {
    int zpb = (tail_rows + groups - 1) / groups;
    if (pair) zpb += zpb & 1;
    work = head;
    int64_t units = 0;
    int longest = 0;
    for (int i = 0; i < kinds; ++i) {
      const int ng = (kind[i].rows + zpb - 1) / zpb;
      work += (double)kind[i].groups * (kind[i].rows + m.item * ng);
      units += kind[i].groups * ng;
      longest = std::max(longest, (kind[i].rows + ng - 1) / ng);
    }
    double time = std::max(zpb + m.item, work / (double)slots + m.end * (zpb + m.item));
    if (tail == 0) {
      const int64_t left = units % slots;
      const double share = (double)((left + cus - 1) / cus * cus) / (double)slots;
      time = (longest + m.item) *
             ((double)(units / slots) + (left ? std::max(m.alone, share) : 0.0));
    }
    time *= 1.0 + ragged * std::min(longest, 100) * 0.01;
    if (best_time < 0.0 || time < best_time * 0.999) {
      best_time = time;
      best.zpb = zpb;
    }
  }
  return best;
}

// Whether a plane, or the planes of a batch, count as ragged: not on 64 bytes in
// rows or segments, and more than the last cache holds.
inline bool ragged_plane(uintptr_t power, int64_t ld, int U) {
  return ((power | (uintptr_t)ld * 4 | (uintptr_t)U * 4) & 63) != 0;
}
constexpr int64_t kCachedPlane = (int64_t)1 << 28;

}  // namespace fdas
