// xbc.h -- inlet/outlet boundaries (Fig. 1) inside passes of several steps
// (block.hip, cascade.hip): columns 0 and nx - 1 emit stored rest equilibria
// in place of their results, as launch_xbc writes them after a single step.
#pragma once

#include "host.h"

namespace lbm {

constexpr int kXbcMaxSteps = 16;  // of a pass

// Stored rest equilibria of the rest, axis and diagonal links at the inlet
// density of each step, and at rho = 1.
template <class T> struct XbcValues {
    T in[kXbcMaxSteps][3], one[3];
};

// The stored value of plane i at a site of wrapped column x whose result was
// f, in step s of the pass.
template <class T> __device__ __forceinline__ T xbc_value(const XbcValues<T>& xb, int s, int i, int ex, int x, int nx, T f)
{
    const int cls = i == 0 ? 0 : (i < 5 ? 1 : 2);
    const T in = xb.in[s][cls], one = xb.one[cls];
    return x == 0 ? (ex < 0 ? one : in) : (x == nx - 1 ? (ex > 0 ? in : one) : f);
}

// The stored rest equilibrium of link class c (rest, axis, diagonal) at
// density rho, with the operations of xbc_kernel.
template <class T, bool SHIFT> T rest_value(int c, double rho, double eqs)
{
    const double w0 = 4.0 / 9.0, w = c == 0 ? w0 : (c == 1 ? 1.0 / 9.0 : 1.0 / 36.0);
    const double r = SHIFT ? rho - 1.0 : rho;
    return (T)(w * r + (c == 0 ? -(1.0 - w0) * r * eqs : w * r * eqs));
}

// The values of a pass of ns steps.
template <class T, bool SHIFT> XbcValues<T> xbc_values(const PassInlet& inlet, int ns)
{
    XbcValues<T> xb;
    for (int c = 0; c < 3; ++c) {
        xb.one[c] = rest_value<T, SHIFT>(c, 1.0, inlet.eqs);
        for (int s = 0; s < kXbcMaxSteps; ++s)
            xb.in[s][c] = rest_value<T, SHIFT>(
                c, inlet_density(inlet.amplitude, inlet.period, inlet.t + (s < ns ? s : 0)), inlet.eqs);
    }
    return xb;
}

}  // namespace lbm
