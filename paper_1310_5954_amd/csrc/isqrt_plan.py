"""Writes isqrt_plan.hpp: the polynomial stages of A^(-1/2) by condition number.

    python paper_1310_5954_amd/csrc/isqrt_plan.py > paper_1310_5954_amd/csrc/isqrt_plan.hpp     (needs mpmath)

A is scaled so that its eigenvalues lie in [1/kappa, 1].  With M_0 = A and
Z_0 = I, a stage takes P = q(M), Z <- P Z, M <- P P M; x = sqrt(eigenvalue of
M) maps to x q(x^2).  A stage's q is the minimax polynomial of that map to 1 on
the interval [l, 1] the previous stages left (Remez exchange), divided by
1 + E (E its error) so that the next interval is again [l', 1]; the last stage
is not divided and ends with E below TOL, so Z = A^(-1/2) to TOL.  The degrees
(in M) are the non-decreasing sequence over {2, 4, 6} (1 too for the last) of
fewest matrix products, after degree 4 while l < 2^-13:
a stage forms its powers and q (0, 1, 2 or 3 products), P Z (none in the first
stage) and, unless it is the last, P (P M) (2).  The last stage's coefficients
are in powers of R = M - I, whose norm is small there.
"""
import sys
from functools import lru_cache

import mpmath as mp
import numpy as np

mp.mp.dps = 50
TOL = mp.mpf("1e-15")
ROWS, MAX_STAGES, MAX_DEG = 105, 11, 6   # row r serves kappa <= 2^(r/2)
POWERS = {1: 0, 2: 1, 4: 2, 6: 3}


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


def last_stage(l, k):
    """Coefficients in R = M - 1, or None when degree k leaves more than TOL."""
    if 1 - l < mp.mpf("1e-12"):  # the binomial series of (1 + R)^(-1/2)
        c = [mp.binomial(mp.mpf(-1) / 2, j) for j in range(k + 1)]
        return c if (1 - l * l) ** (k + 1) < TOL else None
    c, e = minimax(l, k)
    if e > TOL:
        return None
    return [sum(c[i] * mp.binomial(i, j) for i in range(j, k + 1)) for j in range(k + 1)]


def sequences(cost, first=True, least=2, depth=MAX_STAGES):
    """Non-decreasing degree sequences of that many products, the last stage's after a comma."""
    for k in POWERS:
        if POWERS[k] + (0 if first else 1) == cost:
            yield (k,)
    if depth > 1:
        for k in (2, 4, 6):
            spent = POWERS[k] + (0 if first else 1) + 2
            if k >= least and spent < cost:
                for rest in sequences(cost - spent, False, k, depth - 1):
                    yield (k,) + rest


def stages(l, degrees):
    """The stages of that sequence from the interval [l, 1], or None when it leaves more than TOL."""
    got = []
    for k in degrees[:-1]:
        c, e = minimax(l, k)
        if e < mp.mpf("1e-13"):
            return None
        got.append((k, [v / (1 + e) for v in c]))
        l = (1 - e) / (1 + e)
    c = last_stage(l, degrees[-1])
    return None if c is None else got + [(degrees[-1], c)]


def main():
    out = ["// Polynomial stages of A^(-1/2) by condition number: written by isqrt_plan.py, which says how",
           "// they are found.  Row r serves kappa <= 2^(r/2); deg[] ends at the first 0; the last stage's",
           "// coefficients are in powers of M - I, the others' in powers of M.",
           "#pragma once", "", "namespace letkf {", "", f"constexpr int kIsqrtRows = {ROWS};",
           f"constexpr int kIsqrtStages = {MAX_STAGES};", "",
           "struct IsqrtRow {", "  int n, products;", f"  int deg[{MAX_STAGES}];",
           f"  double c[{MAX_STAGES}][{MAX_DEG + 2}];", "};", "",
           "static __device__ const IsqrtRow kIsqrtPlan[kIsqrtRows] = {"]
    prods = 1
    for r in range(ROWS):
        l = mp.mpf(2) ** (mp.mpf(-r) / 4) if r else mp.mpf(2) ** mp.mpf("-0.0001")
        head, got = [], None
        while l < mp.mpf(2) ** -13:  # far from 1 degree 4 gains most per product
            c, e = minimax(l, 4)
            head.append((4, [v / (1 + e) for v in c]))
            l = (1 - e) / (1 + e)
        tail = 1 if head else max(prods, 1)
        while got is None:  # the count does not fall as kappa grows
            got = next((g for g in (stages(l, d) for d in sequences(tail, not head, 4 if head else 2)) if g), None)
            tail += got is None
        prods = tail + (5 * len(head) - 1 if head else 0)
        got = head + got
        deg = [k for k, _ in got] + [0] * (MAX_STAGES - len(got))
        out.append(f"    {{{len(got)}, {prods}, {{{', '.join(map(str, deg))}}}, {{")
        for k, c in got:
            out.append("        {" + ", ".join(mp.nstr(v, 20) for v in c) + "},")
        out.append("    }},")
        print(r, "kappa %.3g" % 2 ** (r / 2), deg, prods, file=sys.stderr, flush=True)
    out += ["};", "", "}  // namespace letkf"]
    print("\n".join(out))


if __name__ == "__main__":
    main()
