"""The adjoint's line formula, checked in FP64 against the two stencils it sums:
with seeds scaled by -1/8, cf = g8_f + gs_f dd_f, cb = g8_b + gs_b dd_b,
s0 = cf - 2 cb + H - F, s1 = cb - 2 cf + H + F, H = -4 (g8_f + g8_b),
F = f (gs_f + gs_b)."""
import numpy as np


def test_scaled_line_adjoint_is_the_sum_of_its_two_stencils():
    rng = np.random.default_rng(8)
    for _ in range(200):
        x = rng.standard_normal(4)   # samples at x-1, x0, x1, x2
        gpf, gpb, gsf, gsb = rng.standard_normal(4)
        gh = (x[2] - x[1]) / 2
        f = 12.0 / 13.0 * gh
        ddf, ddb = (x[1] - 2 * x[2] + x[3]) / 2, (x[2] - 2 * x[1] + x[0]) / 2

        def stencil(gp, gs, dd, slope):   # gradients at a, b, c
            return (0.375 * gp + gs * (dd - slope), 0.75 * gp + gs * (slope - 2 * dd), -0.125 * gp + gs * dd)

        fa, fb, fc = stencil(gpf, gsf, ddf, f)     # (x0, x1, x2)
        ba, bb, bc = stencil(gpb, gsb, ddb, -f)    # (x1, x0, x-1)
        g8f, g8b = -gpf / 8, -gpb / 8
        cf, cb = g8f + gsf * ddf, g8b + gsb * ddb
        F, H = (gsf + gsb) * f, -4 * (g8f + g8b)
        got = (cf - 2 * cb + (H - F), cb - 2 * cf + (H + F), cf, cb)
        assert np.allclose(got, (fa + bb, fb + ba, fc, bc), rtol=0, atol=1e-13)
