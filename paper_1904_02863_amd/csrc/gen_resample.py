#!/usr/bin/env python3
"""Weights of the frequency resampling (writes gw_resample_weights.h).

A phasor g of a rate below NU cycles per node is recovered between uniform
nodes from the 2 P nodes around the point, g(x) ~ sum_t w_t(x) g(t - P + 1),
0 <= x < 1 (one whose rate changes over them, less well near the band's edge).  The weights
are the least-squares ones over the band [-NU, NU]: they minimise
    int_{-NU}^{NU} |e^{2 pi i nu x} - sum_t w_t e^{2 pi i nu (t - P + 1)}|^2 dnu,
i.e. solve the normal equations G w = b with G_ij = sinc(2 NU (i - j)) and
b_i = sinc(2 NU (i - x)).  G is ill-conditioned (that is what makes the error
small), so they are solved with 70 digits and a ridge of 1e-33, which keeps
the weights' sum of magnitudes near 2.  Each weight is a smooth function of x
and is written as a polynomial in s = 2 x - 1, interpolated at Chebyshev
points, so that the kernels can form the weights of any bin spacing.  The
weights are mirror images, w_t(s) = w_{TAPS - 1 - t}(-s), so the header holds
those of the lower half, and one evaluation of their even and odd parts gives
a pair: w_t = E + s O, w_{TAPS - 1 - t} = E - s O with polynomials E, O in s^2.

    python gen_resample.py            # writes the header
    python gen_resample.py --check    # prints the error of the double evaluation
"""
import os
import sys

import mpmath as mp
import numpy as np

mp.mp.dps = 70
P = 16                      # nodes on each side
TAPS = 2 * P
NU = mp.mpf(1) / 5          # band edge, cycles per node
DEGREE = 13                 # of the polynomials in s
RIDGE = mp.mpf(10) ** -33
OUT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "gw_resample_weights.h")


def sinc(d):
    return mp.mpf(1) if d == 0 else mp.sin(2 * mp.pi * NU * d) / (2 * mp.pi * NU * d)


def weights_at(xs):
    """Least-squares weights [len(xs)][TAPS] as mpf."""
    nodes = [mp.mpf(t - P + 1) for t in range(TAPS)]
    g = mp.matrix(TAPS, TAPS)
    for i in range(TAPS):
        for j in range(TAPS):
            g[i, j] = sinc(nodes[i] - nodes[j]) + (RIDGE if i == j else 0)
    inv = g ** -1
    out = []
    for x in xs:
        b = mp.matrix([sinc(n - x) for n in nodes])
        out.append(list(inv * b))
    return out


def polynomials():
    """Coefficients [TAPS][DEGREE + 1] (lowest power of s first) as floats."""
    n = DEGREE + 1
    s = [mp.cos(mp.pi * (2 * i + 1) / (2 * n)) for i in range(n)]
    w = weights_at([(si + 1) / 2 for si in s])
    vand = mp.matrix(n, n)
    for i in range(n):
        for j in range(n):
            vand[i, j] = s[i] ** j
    inv = vand ** -1
    return [[float(v) for v in inv * mp.matrix([w[i][t] for i in range(n)])] for t in range(TAPS)]


def evaluate(coef, x):
    """Weights [len(x)][TAPS] in double from the lower half's coefficients, as
    the kernels form them."""
    c = np.asarray(coef)[:P]
    s = 2.0 * np.asarray(x, dtype=np.float64)[:, None] - 1.0
    z = s * s
    even = np.broadcast_to(c[:, DEGREE - 1], (s.shape[0], P)).copy()
    odd = np.broadcast_to(c[:, DEGREE], (s.shape[0], P)).copy()
    for j in range(DEGREE - 3, -1, -2):
        even = even * z + c[:, j]
        odd = odd * z + c[:, j + 1]
    return np.hstack([even + s * odd, (even - s * odd)[:, ::-1]])


def band_error(coef, nu_max=float(NU), n_x=97, n_nu=120):
    """Worst |e^{2 pi i nu x} - sum w e^{..}| over x in [0, 1), |nu| <= nu_max,
    and the largest sum of |w| (the sums in extended precision)."""
    x = np.arange(n_x) / n_x
    w = evaluate(coef, x).astype(np.longdouble)
    two_pi = 2 * np.longdouble("3.14159265358979323846264338327950288")
    t = np.arange(TAPS) - P + 1
    worst = 0.0
    for nu in np.linspace(0.0, nu_max, n_nu).astype(np.longdouble):
        d = two_pi * nu * (t[None, :] - x[:, None].astype(np.longdouble))
        c = (w * np.cos(d)).sum(1) - 1
        s = (w * np.sin(d)).sum(1)
        worst = max(worst, float(np.sqrt(c * c + s * s).max()))
    return worst, float(np.abs(w).sum(1).max())


def header(coef) -> str:
    """The text of gw_resample_weights.h."""
    e, _ = band_error(coef)
    rows = []
    for j in range(DEGREE + 1):
        vals = [repr(coef[t][j]) for t in range(P)]
        lines = [", ".join(vals[i:i + 4]) for i in range(0, P, 4)]
        rows.append("    {" + ", \\\n     ".join(lines) + "}")
    return ("// Written by gen_resample.py.  Weights of the frequency resampling: weight t (node\n"
            f"// offset t - {P - 1}) of a point a fraction x of a node spacing past node 0 is the\n"
            "// polynomial sum_j GW_RESAMPLE_COEF[j][t] s^j, s = 2 x - 1.  Recovers phasors of a\n"
            f"// constant rate of up to {float(NU)} cycles per node to {e:.1e} (worst case over the band).\n"
            "#pragma once\n\n"
            f"#define GW_RESAMPLE_HALF {P}\n#define GW_RESAMPLE_TAPS {TAPS}\n"
            f"#define GW_RESAMPLE_DEGREE {DEGREE}\n#define GW_RESAMPLE_BAND {float(NU)!r}\n"
            "#define GW_RESAMPLE_COEF_VALUES \\\n" + ", \\\n".join(rows) + "\n")


def main():
    coef = polynomials()
    e, l1 = band_error(coef)
    print(f"taps {TAPS}, band edge {float(NU)} cycles per node, degree {DEGREE}: worst error {e:.2e}, "
          f"largest sum of |w| {l1:.3f}")
    if "--check" not in sys.argv:
        with open(OUT, "w") as fh:
            fh.write(header(coef))


if __name__ == "__main__":
    main()
