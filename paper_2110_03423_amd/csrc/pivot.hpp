// Pivots of a factorisation that are looked at when all are done.
#pragma once

namespace rsvd {

// From r = R[c][c], the rounded root of a pivot d: was d above thr?  True says so for certain, whatever r's rounding (the root is good to 2 ulp, its square to 5
// roundings); within a few roundings of the threshold it is false, and the elimination is done again with a look at each pivot itself, which decides.
// So the columns that are dropped or set aside do not depend on which of the two was done first.
constexpr bool pivot_surely_above(double r, double thr) { return r * r > thr * (1.0 + 16 * 2.220446049250313e-16); }

}  // namespace rsvd
