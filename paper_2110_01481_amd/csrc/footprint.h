// Areas of trapezoids, shared by the strip-model projectors: the footprint of a unit pixel on
// the detector (boxes of p and q = max and min(|cos|, |sin|) convolved) for the transposes, the
// extent of a strip along a band of pixels for the forward projector.
#pragma once

#include "geometry.h"

namespace abg {
namespace {

// A trapezoid of unit area, the convolution of boxes of widths a >= b >= 0 (a > 0): flat
// within h0 = (a - b)/2 of its centre, zero beyond h1 = (a + b)/2. operator()(t) is its area
// between the centre and t, an odd function:
//     t/a up to h0, less (|t| - h0)^2 / (2 a b) beyond, 1/2 from h1 on.
// Differences of it over consecutive edges are the areas between them, so n parts cost
// n - 1 evaluations of six instructions.
template <typename T> struct HalfArea {
    T h0, h1, inva, i2ab;
    HalfArea() = default;
    __device__ HalfArea(double a, double b)
        : h0(T(0.5 * (a - b))), h1(T(0.5 * (a + b))), inva(T(1.0 / a)),
          i2ab(b > 0.0 ? T(fmin(0.5 / (a * b), 1e30)) : T(0))
    {
    }
    __device__ T operator()(T t) const
    {
        const T d = fmin(fabs(t), h1), m = fmax(d - h0, T(0));
        return copysign(fma(-m * i2ab, m, d * inva), t);
    }
};

}  // namespace
}  // namespace abg
