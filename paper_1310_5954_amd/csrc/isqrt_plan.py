"""Writes isqrt_plan.hpp: the polynomial stages of A^(-1/2) by condition number.

    python paper_1310_5954_amd/csrc/isqrt_plan.py > paper_1310_5954_amd/csrc/isqrt_plan.hpp     (needs mpmath)

A is scaled so that its eigenvalues lie in [1/kappa, 1].  With M_0 = A and
Z_0 = I, a stage takes P = q(M), Z <- P Z, M <- P P M; x = sqrt(eigenvalue of
M) maps to x q(x^2).  A stage's q is the minimax polynomial of that map to 1 on
the interval [l, 1] the stages before it left (Remez exchange), divided by
1 + E (E its error), so that the next interval is again [l', 1], less TOP, so
that no rounding takes an eigenvalue past 1, where the next stages' slopes (50
and more) would carry it away.  An eigenvalue below l^2 stays in (0, 1) and
gains at least as much as one at l^2, so a stage for too small a kappa costs
further stages and nothing else.

The last stage maps to 1 within TOL without the division.  Its polynomials are
in powers of R = M - I, of degree 2, 4 or 6, for ||R|| <= kIsqrtRho; the
kernels choose by the bound ||R^2||_F^(1/2) >= ||R||, up to m^(1/4) times the
norm, so the stages before it aim at a MARGIN-th of that.

kIsqrtPlan: row r serves kappa <= 2^(r/2) (row 0: 1.05) by stages of degree 4,
one at least, and the last.  A stage forms M^2 and q (2 products in all; 1 and 3
for degrees 2 and 6), P Z (not in the first stage) and, unless it is the last,
P (P M) (2).  Degree 4 gains most per product until little is left to gain;
stages of degree 2 or 6 before the last would save a product here and there,
at a branch per stage whose registers the kernel does not have, and degree 6
at a digit (its coefficients sum to 3e4 in size, those of degree 4 to 1e3).

kIsqrtStage4: the same stages singly, entry i - 1 for kappa <= 2^(i/4); `next` is
the entry number of the interval it leaves, 0 where that is near enough to 1
for a last stage of degree 4.
"""
import sys
from functools import lru_cache

import mpmath as mp
import numpy as np

mp.mp.dps = 50
TOL, TOP = mp.mpf("2e-16"), mp.mpf("1e-10")
ROWS, MAX_STAGES, MAX_DEG, ENTRIES, MARGIN = 105, 12, 6, 208, 3
PRODUCTS = {2: 1, 4: 2, 6: 3}  # to form q(M)
RHO = {2: mp.mpf("2.7e-5"), 4: mp.mpf("3.3e-3"), 6: mp.mpf("2.5e-2")}


@lru_cache(maxsize=None)
def minimax(l, k):
    """q of degree k in x^2 that minimises max |1 - x q(x^2)| on [l, 1], and that maximum."""
    n = k + 1
    cheb = [(1 - mp.cos(mp.pi * j / n)) / 2 for j in range(n + 1)]
    x = [l ** (1 - c) if l < mp.mpf("0.3") else l + (1 - l) * c for c in cheb]
    last = None
    for _ in range(60):
        rows = mp.matrix(n + 1, n + 1)
        for r in range(n + 1):
            for i in range(n):
                rows[r, i] = x[r] ** (2 * i + 1)
            rows[r, n] = (-1) ** r
        s = mp.lu_solve(rows, mp.matrix([1] * (n + 1)))
        c, e = [s[i] for i in range(n)], abs(s[n])
        poly = [(2 * i + 1) * c[i] for i in range(n)]  # p' in t = x^2
        new = [l]
        w = mp.mpf(1) if l < mp.mpf("0.3") else 1 - l * l  # first guesses in u, t = (1 - w) + w u
        inu = [w ** j * sum(poly[i] * mp.binomial(i, j) * (1 - w) ** (i - j) for i in range(j, n)) for j in range(n)]
        for u in sorted(np.real(np.roots([float(v / max(map(abs, inu))) for v in inu[::-1]]))):
            t = (1 - w) + w * mp.mpf(float(u))
            for _n in range(8):
                t -= mp.polyval(poly[::-1], t) / mp.polyval([j * poly[j] for j in range(1, n)][::-1], t)
            new.append(mp.sqrt(t))
        x = new + [mp.mpf(1)]
        assert all(x[j] < x[j + 1] for j in range(n)), (l, k)
        if last is not None and abs(e - last) <= e * mp.mpf(10) ** -12:
            break
        last = e
    return c, max(abs(1 - sum(c[i] * t ** (2 * i + 1) for i in range(n))) for t in x)


@lru_cache(maxsize=None)
def last_stage(k):
    """Coefficients in R = M - 1 for eigenvalues of R in [-rho, 0]."""
    c, e = minimax(mp.sqrt(1 - RHO[k]), k)
    assert e <= TOL, (k, e)
    return [sum(c[i] * mp.binomial(i, j) for i in range(j, k + 1)) for j in range(k + 1)]


def stage(l, k):
    """Coefficients of a stage from [l, 1], and the l it leaves."""
    c, e = minimax(l, k)
    f = (1 - TOP) / (1 + e)
    return [v * f for v in c], (1 - e) * f


def last_degree(l, degrees=(2, 4, 6)):
    return next((k for k in degrees if 1 - l * l <= RHO[k] / MARGIN), None)


def sequence(l):
    """The stages from [l, 1] as (degree, coefficients), and their products."""
    got, x = [], l
    while True:
        c, x = stage(x, 4)
        got.append((4, c))
        end = last_degree(x)
        if end:
            return got + [(end, last_stage(end))], 5 * len(got) - 1 + PRODUCTS[end] + 1


def main():
    out = ["// Polynomial stages of A^(-1/2) by condition number: written by isqrt_plan.py, which says how",
           "// they are found.  Row r of kIsqrtPlan serves kappa <= 2^(r/2); deg[] ends at the first 0; the last",
           "// stage's coefficients are in powers of M - I, the others' in powers of M.  Entry i - 1 of",
           "// kIsqrtStage4 serves kappa <= 2^(i/4) and leaves the interval of entry `next` (0: the last stage's).",
           "#pragma once", "", "namespace letkf {", "", f"constexpr int kIsqrtRows = {ROWS};",
           f"constexpr int kIsqrtStages = {MAX_STAGES};", f"constexpr int kIsqrtEntries = {ENTRIES};", "",
           "struct IsqrtRow {", "  int n, products;", f"  int deg[{MAX_STAGES}];",
           f"  double c[{MAX_STAGES}][{MAX_DEG + 2}];", "};", "struct IsqrtStage {", "  int next;", "  double c[5];", "};", "",
           "static __device__ const IsqrtRow kIsqrtPlan[kIsqrtRows] = {"]
    for r in range(ROWS):
        l = mp.mpf(2) ** (mp.mpf(-r) / 4) if r else 1 / mp.sqrt(mp.mpf("1.05"))
        got, products = sequence(l)
        deg = [k for k, _ in got] + [0] * (MAX_STAGES - len(got))
        out.append(f"    {{{len(got)}, {products}, {{{', '.join(map(str, deg))}}}, {{")
        for k, c in got:
            out.append("        {" + ", ".join(mp.nstr(v, 20) for v in c) + "},")
        out.append("    }},")
        print(r, "kappa %.3g" % 2 ** (r / 2), deg, products, file=sys.stderr, flush=True)
    out += ["};", "", "static __device__ const IsqrtStage kIsqrtStage4[kIsqrtEntries] = {"]
    for i in range(1, ENTRIES + 1):
        c, low = stage(mp.mpf(2) ** (mp.mpf(-i) / 8), 4)
        nxt = 0 if last_degree(low, (4,)) else int(mp.ceil(-8 * mp.log(low, 2)))
        assert nxt < i
        out.append(f"    {{{nxt}, {{" + ", ".join(mp.nstr(v, 20) for v in c) + "}},")
    out += ["};", "", "// the last stage: degree 2, 4, 6 for ||M - I|| <= kIsqrtRho",
            "constexpr double kIsqrtRho[3] = {" + ", ".join(mp.nstr(RHO[k], 6) for k in (2, 4, 6)) + "};",
            "static __device__ const double kIsqrtLast[3][7] = {"]
    for k in (2, 4, 6):
        out.append("    {" + ", ".join(mp.nstr(v, 20) for v in last_stage(k)) + "},")
    out += ["};", "", "}  // namespace letkf"]
    print("\n".join(out))


if __name__ == "__main__":
    main()
