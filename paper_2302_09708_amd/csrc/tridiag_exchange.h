// Which workgroups of the tridiagonalisation (tridiag.hip) take part in the exchange of a
// column.  Plain constexpr functions: the kernel uses them, and a host model of the exchange
// (tests/tridiag_exchange_model.cpp) runs them under every delay of a workgroup.
//
// Row j lives in workgroup j % groups, columns go from n - 1 down to 1, and column m has the
// active rows 0 .. m - 1.  Its slots are in set (n - m) % 2, so column m - 2 writes over them.
#pragma once

namespace chefsi {

constexpr int td_set(int n, int m) { return (n - m) & 1; }

// A workgroup publishes its active rows' slots of column m.
constexpr bool td_publishes(int me, int m) { return me < m; }

// It reads all of column m's slots only if it also publishes column m - 1: whoever writes
// column m - 2 has read column m - 1 whole, and so knows that every reader of column m is done
// with the slots that it writes over.  A workgroup that does not read a column has no work left
// and leaves; workgroup 0, which writes the results, stays to the end (row 0 is active in
// every column, and behind column 1 no slot is written any more).
constexpr bool td_reads(int me, int m) { return me == 0 || td_publishes(me, m - 1); }

}  // namespace chefsi
