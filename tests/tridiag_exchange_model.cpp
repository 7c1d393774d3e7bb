// Host model of the exchange of the tridiagonalisation (csrc/tridiag.hip) under any delay.
//
// G workgroups publish their active rows' slots of a column and then read all active slots of
// it, over and over until one pass finds this column's number in every slot; two sets of slots
// alternate.  Prints "rule groups n runs stuck": the runs that end with a workgroup waiting for
// a number that nobody will write again.
//   rule 0: the kernel's (td_reads);  1: every workgroup reads every column;
//   rule 2: a workgroup reads every column in which it has a row.
// Delays: one workgroup is stopped at a column before its publication, before its first look or
// in the middle of one while the others go as far as they can, then goes on (every workgroup,
// column and place); and random schedules in which workgroups sleep for random stretches.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "tridiag_exchange.h"

namespace {

bool reads(int rule, int me, int m) {
  return rule == 0 ? chefsi::td_reads(me, m) : (rule == 1 ? true : me == 0 || me < m);
}

struct Model {
  int rule, groups, n;
  std::vector<int> slot[2];                    // the column number of every slot's content
  std::vector<int> column, next, row, at;      // per workgroup: m, the phase below, its next row, its next look
  enum Phase { Publish, Read, Gone };

  Model(int rule_, int groups_, int n_) : rule(rule_), groups(groups_), n(n_) {
    slot[0].assign(n, 0);
    slot[1].assign(n, 0);
    column.assign(groups, n - 1);
    next.assign(groups, Publish);
    at.assign(groups, 0);
    row.resize(groups);
    for (int q = 0; q < groups; ++q) row[q] = q;
  }

  // One action of workgroup q: a slot written or looked at.  False when it is gone, or has just
  // looked in vain (its pass starts anew).
  bool act(int q) {
    const int m = column[q], set = chefsi::td_set(n, m);
    if (next[q] == Gone) return false;
    if (next[q] == Publish) {
      if (row[q] < m) {
        slot[set][row[q]] = n - m;
        row[q] += groups;
      }
      if (row[q] >= m) {
        next[q] = reads(rule, q, m) ? Read : Gone;
        at[q] = 0;
      }
      return true;
    }
    if (slot[set][at[q]] != n - m) {
      at[q] = 0;
      return false;
    }
    if (++at[q] == m) {
      column[q] = m - 1;
      row[q] = q;
      next[q] = m > 1 ? Publish : Gone;
    }
    return true;
  }

  // All but `stopped` until none of them gets on: a publication or a whole column read (looks
  // that end in vain are no progress).
  void settle(int stopped) {
    for (bool any = true; any;) {
      any = false;
      for (int q = 0; q < groups; ++q) {
        if (q == stopped || next[q] == Gone) continue;
        for (;;) {
          const int m = column[q], was = next[q];
          bool more = true;
          while (more && column[q] == m && next[q] == was) more = act(q);
          if (!more || next[q] == Gone) {
            any = any || more;
            break;
          }
          any = true;
        }
      }
    }
  }

  bool stuck() {
    settle(-1);
    for (int q = 0; q < groups; ++q)
      if (next[q] != Gone) return true;
    return false;
  }
};

}  // namespace

int main(int argc, char** argv) {
  const int rule = std::atoi(argv[1]), groups = std::atoi(argv[2]), n = std::atoi(argv[3]);
  long runs = 0, stuck = 0;
  for (int q = 0; q < groups; ++q)
    for (int m = n - 1; m >= 1; --m)
      for (int place = 0; place < 3; ++place) {
        Model w(rule, groups, n);
        // everyone together up to the place where q stops
        auto there = [&] {
          if (w.next[q] == Model::Gone || w.column[q] < m) return true;
          if (w.column[q] > m) return false;
          return place == 0 || (w.next[q] == Model::Read && (place == 1 || w.at[q] > m / 2 || m == 1));
        };
        while (!there())
          for (int p = 0; p < groups && !there(); ++p) w.act(p);
        w.settle(q);
        ++runs;
        stuck += w.stuck();
      }
  std::mt19937 rng(7u + 31u * groups + n);
  for (int k = 0; k < 200; ++k) {
    Model w(rule, groups, n);
    std::vector<int> asleep(groups, 0);
    for (int t = 0; t < 40 * n * groups; ++t) {
      const int q = (int)(rng() % groups);
      if (asleep[q] > 0)
        --asleep[q];
      else if (rng() % (4 * n) == 0)
        asleep[q] = (int)(rng() % (8 * n));
      else
        for (int i = 0; i < 1 + (int)(rng() % n) && w.act(q); ++i) {
        }
    }
    ++runs;
    stuck += w.stuck();
  }
  std::printf("%d %d %d %ld %ld\n", rule, groups, n, runs, stuck);
  return 0;
}
