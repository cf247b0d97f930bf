// Host-logic check of the collision's coefficients (make_coef in host.h),
// built with g++ by test_coefficients.py: the sums that conserve mass and
// momentum close exactly, and every coefficient is its formula rounded to a
// few units. Sums in long double, which holds them exactly.
#include <cstdio>

#include "host.h"

namespace lbm {
int moments_blocks(const Geom&) { return 1; }  // declared in host.h, not used here
}

static int fails = 0;

template <class C> void check(const lbm::CoefSet<C>& k, double tau, double c2, int model)
{
    using D = long double;
    const D om = 1 / (D)tau, sh = lbm::eq_shift(c2, model), eps = sizeof(C) == 4 ? 0x1p-24L : 0x1p-53L;
    auto bad = [&](const char* what, D v) {
        if (++fails <= 20) std::printf("FAIL %s %.3Le: %d bytes tau %.17g c2 %.17g model %d\n", what, v, (int)sizeof(C), tau, c2, model);
    };
    auto zero = [&](const char* what, D v) {
        if (v != 0) bad(what, v);
    };
    zero("momentum", (D)k.om1 + 3 * (D)k.w3 - 1);
    zero("mass", (D)k.om1 + (D)k.a0 + 4 * (D)k.a1 + 4 * (D)k.a2 - 1);
    zero("mass of j.u", (D)k.b0 + 4 * (D)k.b1 + 4 * (D)k.b2 + 2 * (D)k.t45);
    zero("mass of the constant", (D)k.z0 + 4 * (D)k.z1 + 4 * (D)k.z2);
    zero("t9", (D)k.t9 - (D)k.t45 / 2);
    // om1 lies within three half units of 1 (eps = half a unit of 1) of its
    // formula; the others follow it, each with roundings of its own of at
    // most two units of 1
    auto near = [&](const char* what, C v, D f) {
        if (std::fabs((D)v - f) > 3 * eps) bad(what, (D)v - f);
    };
    near("om1", k.om1, 1 - om);
    const D rel = 1 - (D)k.om1, w0 = 4 / 9.0L, w1 = 1 / 9.0L, w2 = 1 / 36.0L, e0 = -1.25L * sh;
    near("w3", k.w3, rel * 3 * w1);
    near("a0", k.a0, rel * w0 * (1 + e0));
    near("a1", k.a1, rel * w1 * (1 + sh));
    near("a2", k.a2, rel * w2 * (1 + sh));
    near("b0", k.b0, -1.5L * rel * w0);
    near("b1", k.b1, -1.5L * rel * w1);
    near("b2", k.b2, 3 * rel * w2);
    near("t45", k.t45, 4.5L * rel * w1);
    near("z0", k.z0, om * w0 * e0);
    near("z1", k.z1, om * w1 * sh);
    if (model == LBM_MODEL_FORCING) zero("pressure", 6 * (D)k.a1 + 12 * (D)k.a2 - rel);
    else near("pressure", k.a1, (rel * (D)c2 - 4 * (D)k.a2) / 2);
    if (!(k.a0 >= 0 && k.a1 > 0 && k.a2 > 0)) bad("sign", 0);
}

int main()
{
    // tau from just above 1/2 to 50 and at round values; c2 over each model's range
    for (int n = 0; n < 4000; ++n) {
        const double tau = n < 3000 ? 0.5001 + n * 0.00050731 : (n < 3900 ? 2.0 + (n - 3000) * 0.05331 : 0.55 + (n - 3900) / 64.0);
        for (int m = 0; m < 12; ++m) {
            const double c = 0.04 + m * 0.0507;
            const double a = m == 0 ? 1.0 / 3.0 : 0.04 + m * 0.0508;  // below 0.6
            for (int model : {LBM_MODEL_FORCING, LBM_MODEL_EQUILIBRIUM}) {
                const double v = model == LBM_MODEL_FORCING ? c : a;
                check(lbm::make_coef(tau, v, model).d, tau, v, model);
                check(lbm::make_coef(tau, v, model).f, tau, v, model);
            }
        }
    }
    std::puts(fails ? "FAILED" : "coefficients ok");
    return fails != 0;
}
