"""The analysis perturbations X' W of the FP64 path against extended precision,
where the state lives: W's largest eigenvalue belongs to the vector of ones,
which X' annihilates, so an error of T measured as a whole says nothing of it.

The reference is W in numpy's long double (Cholesky and one-sided Jacobi of
A = (m-1)/rho I + C, C from the long double ensemble).  The bound is what
double precision makes of T = W + wbar 1^T on the same domains by Cholesky + SVD,
four times over: both carry the rounding of C and of the sum, and two roundings
of the same C scatter by that much; 1e-14 is the floor, the rounding of the
products themselves.  R^-1 is
scaled up to 1e6: kappa(A) then reaches 1e11, but off the vector of ones it
stays that of C wherever a domain has more slopes than members."""
import numpy as np
import pytest

from paper_1310_5954_amd import FP64, Filter, Problem
from workload.configs import CONFIGS, build_case

pytestmark = pytest.mark.gpu
L = np.longdouble


def inverse_root(A):
    """A^(-1/2) in long double: Cholesky, one-sided Jacobi in round-robin order."""
    m0 = len(A)
    m = m0 + m0 % 2
    chol = np.zeros((m0, m0), dtype=L)
    for j in range(m0):
        v = A[j:, j] - chol[j:, :j] @ chol[j, :j]
        chol[j:, j] = v / np.sqrt(v[0])
    B = np.eye(m, dtype=L)
    B[:m0, :m0] = chol
    for _ in range(30):
        big, order = 0.0, np.arange(m)
        for _round in range(m - 1):
            p, q = order[:m // 2], order[m // 2:][::-1]
            bp, bq = B[:, p], B[:, q]
            al, be, g = (bp * bp).sum(0), (bq * bq).sum(0), (bp * bq).sum(0)
            big = max(big, float(np.max(np.abs(g) / np.sqrt(al * be))))
            z = (be - al) / np.where(g == 0, 1, 2 * g)
            t = np.where(g == 0, 0, np.where(z >= 0, 1, -1) / (np.abs(z) + np.sqrt(1 + z * z)))
            c = 1 / np.sqrt(1 + t * t)
            B[:, p], B[:, q] = c * (bp - t * bq), c * (t * bp + bq)
            order = np.concatenate([order[:1], order[-1:], order[1:-1]])
        if big < 1e-17:
            break
    lam = (B * B).sum(0)
    return ((B / lam) @ (B / np.sqrt(lam)).T)[:m0, :m0]


def domain(case, l, y, kind):
    """X' (both instants), A and b of a domain, in that type."""
    X = case.X0.astype(kind)
    na, m = case.n_act, case.m
    o, e = case.dmap.obs(l), case.dmap.est(l)
    rows = np.concatenate([o, case.n_sub + o])
    taper = np.concatenate([case.dmap.taper(l)] * 2).astype(kind)
    Y = np.stack([(case.D.val[a:b, None].astype(kind) * X[:na][case.D.col[a:b]]).sum(0)
                  for a, b in zip(case.D.rowptr[rows], case.D.rowptr[rows + 1])])
    d = y[rows] - Y.mean(1)
    Y = Y - Y.mean(1)[:, None]
    r = taper * case.r_inv[rows].astype(kind)
    Xp = X - X.mean(1)[:, None]
    A = np.eye(m, dtype=kind) * kind((m - 1) / case.inflation) + (np.sqrt(r)[:, None] * Y).T @ (np.sqrt(r)[:, None] * Y)
    return Xp[np.concatenate([e, na + e])], A, Y.T @ (r * d)


# (configuration, changes to it, members, one global domain): fewer and more
# slopes than members, every tile count of the kernels, m > 128
CASES = [(1, {}, 16, False), (2, dict(lenslets=20), 31, False), (2, dict(lenslets=20, window=6, taper=False), 48, False),
         (3, dict(lenslets=24), 64, False), (2, dict(lenslets=20, window=6, taper=False), 75, False),
         (3, dict(lenslets=24, taper=False), 100, False), (2, dict(lenslets=20, window=6, taper=False), 128, False),
         (2, dict(lenslets=16), 150, True), (2, dict(lenslets=32), 197, True)]


@pytest.mark.parametrize("config,change,m,whole", CASES)
@pytest.mark.parametrize("scale", [1.0, 1e4, 1e6])
def test_perturbations_as_accurate_as_cholesky_and_svd(config, change, m, whole, scale):
    case = build_case(dict(CONFIGS[config], **change), m=m, global_map=whole)
    case.r_inv = case.r_inv * scale
    f = Filter(Problem.from_case(case), case.X0, precision=FP64, debug=True)
    y = case.slopes(0)
    f.analyse(y)
    n = case.dmap.n_domains
    got, want = {}, {}  # by whether a domain has slopes for every direction
    for l in sorted({0, n // 3, n // 2, n - 1}):
        Xp, A, b = domain(case, l, y, L)
        Z = inverse_root(A)
        wbar = (Z @ (Z @ b)).astype(float)
        ref = Xp @ Z
        ref = np.sqrt(L(m - 1)) * (ref - ref.mean(1)[:, None])

        def error(T):
            x = Xp @ np.asarray(T, dtype=L)
            x = x - x.mean(1)[:, None]  # without the mean's update and what X' 1 = 0 leaves
            return float(np.linalg.norm((x - ref).astype(float)) / np.linalg.norm(ref.astype(float)))
        Ad = domain(case, l, y, np.float64)[1]
        u, s, _ = np.linalg.svd(np.linalg.cholesky(Ad))
        full = 2 * len(case.dmap.obs(l)) >= m - 1
        want[full] = max(want.get(full, 0.0), error(np.sqrt(m - 1) * (u / s) @ u.T + wbar[:, None]))
        got[full] = max(got.get(full, 0.0), error(f.debug_domain(l)["T"]))
    assert f.unconverged() == 0
    f.close()
    for full in got:
        print(f"m {m} scale {scale:g} {'more' if full else 'fewer'} slopes than members: {got[full]:.2e}, "
              f"Cholesky + SVD {want[full]:.2e}")
        assert got[full] < 4 * want[full] + 1e-14
