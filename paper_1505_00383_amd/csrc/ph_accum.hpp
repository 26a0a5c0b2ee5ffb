// ph_accum.hpp -- running sums of L-limb values (the tracker's sum of an
// equation's term values).
//
// Every limb has its own running sum; the rounding error of each addition joins
// the next limb, and a guard limb behind the last one takes what the last one
// cannot hold.  The limbs are not renormalised between the additions, so what a
// term adds to the dependency chain is one addition per limb, where a normalised
// addition is a chain of thirteen (double double).  Limb 1 and those behind it
// grow with the terms, so their additions are error free too; only the guard limb,
// an order eps below the result's last one, is summed with rounding.  Double
// double takes the errors of the second limb by FastTwoSum: the first limb's
// error is mostly the larger one and the running sum nearly always; where they
// are not, one rounding of that limb is lost, as a normalised addition loses two.
// Median error of the sum of 130 values of size 1: quad double 4e-62 without the
// guard limb, 3e-64 by normalised additions, 5e-66 here; double double 5e-31,
// 1.9e-31 and 4.5e-32.  20000 paths of 16 systems in double double: 119 ms without
// the guard limb, 122 ms here, 128 ms with TwoSum throughout (7e-33).
#pragma once

#include "ph_arith.hpp"

namespace ph {

template <int L>
struct Acc {
    double v[L == 1 ? 1 : L + 1];
};

template <int L>
PH_HD Acc<L> acc_zero()
{
    Acc<L> s;
    for (double &x : s.v) x = 0.0;
    return s;
}

template <int L>
PH_HD void acc_add(Acc<L> &s, const R<L> &u)
{
    if constexpr (L == 1) {
        s.v[0] += u.v[0];
    } else if constexpr (L == 2) {
        double e, f, g;
        two_sum(s.v[0], u.v[0], s.v[0], e);
        fast_two_sum(e, u.v[1], e, f);
        fast_two_sum(s.v[1], e, s.v[1], g);
        s.v[2] += f + g;
    } else {
        double e0, e1, f, g, h, k, p, q, r, w;
        two_sum(s.v[0], u.v[0], s.v[0], e0);
        two_sum(s.v[1], u.v[1], s.v[1], e1);
        two_sum(s.v[1], e0, s.v[1], f);
        two_sum(s.v[2], u.v[2], s.v[2], g);
        two_sum(s.v[2], e1, s.v[2], h);
        two_sum(s.v[2], f, s.v[2], k);
        two_sum(s.v[3], u.v[3], s.v[3], p);
        two_sum(s.v[3], g, s.v[3], q);
        two_sum(s.v[3], h, s.v[3], r);
        two_sum(s.v[3], k, s.v[3], w);
        s.v[4] += (p + q) + (r + w);
    }
}

// The sum as L limbs.
template <int L>
PH_HD R<L> acc_value(const Acc<L> &s)
{
    if constexpr (L == 1) {
        return R<1>{{s.v[0]}};
    } else if constexpr (L == 2) {
        double a, b;
        R<2> r;
        two_sum(s.v[1], s.v[2], a, b);
        two_sum(s.v[0], a, r.v[0], r.v[1]);
        r.v[1] += b;
        two_sum(r.v[0], r.v[1], r.v[0], r.v[1]);
        return r;
    } else {
        // limbs may overlap and cancel against each other: three passes
        // leave the sum in the leading limbs
        double a[5];
#pragma unroll
        for (int l = 0; l < 5; ++l) a[l] = s.v[l];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            two_sum(a[3], a[4], a[3], a[4]);
            two_sum(a[2], a[3], a[2], a[3]);
            two_sum(a[1], a[2], a[1], a[2]);
            two_sum(a[0], a[1], a[0], a[1]);
        }
        return R<4>{{a[0], a[1], a[2], a[3] + a[4]}};
    }
}

}  // namespace ph
