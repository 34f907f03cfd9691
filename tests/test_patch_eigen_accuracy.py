"""Host check: the patch eigenpairs are those of the 1-D patch matrices to the
rounding of their entries, in extended precision (np.longdouble).  The direct
smoothers solve for whole values with them, so an error here is one of x."""
import numpy as np
import pytest

from paper_2405_18982_amd import dgmg, inputs

LD = np.longdouble
pytestmark = pytest.mark.skipif(np.finfo(LD).eps > 1e-18, reason="needs an extended long double")


def legendre(m, x):
    """P_m(x) and P_m'(x)."""
    p0, p1, d0, d1 = LD(1), x, LD(0), LD(1)
    for j in range(2, m + 1):
        p0, p1, d0, d1 = p1, ((2 * j - 1) * x * p1 - (j - 1) * p0) / LD(j), d1, d0 + (2 * j - 1) * p1
    return p1, d1


def newton(x, step):
    for _ in range(30):
        x = x - step(x)
    return x


def cell_matrices(k):
    """Mass, stiffness and end derivatives of Q_k on [0, 1]."""
    n = k + 1

    def lobatto(x):
        p, d = legendre(k, x)
        return d * (1 - x * x) / (2 * x * d - k * n * p)

    def gauss(x):
        p, d = legendre(n, x)
        return p / d

    inner = [newton(LD(-np.cos(np.pi * j / k)), lobatto) for j in range(1, k)]
    nodes = (np.array([LD(-1)] + inner + [LD(1)]) + 1) / 2
    g = np.array([newton(LD(-np.cos(np.pi * (i + 0.75) / (n + 0.5))), gauss) for i in range(n)])
    w = np.array([1 / ((1 - x * x) * legendre(n, x)[1] ** 2) for x in g])  # on [0, 1]
    g = (g + 1) / 2

    def basis(x):
        V, G = np.zeros((len(x), n), LD), np.zeros((len(x), n), LD)
        for j in range(n):
            oth = [m for m in range(n) if m != j]
            den = np.prod(nodes[j] - nodes[oth])
            for i, y in enumerate(x):
                V[i, j] = np.prod(y - nodes[oth]) / den
                G[i, j] = sum(np.prod([y - nodes[m] for m in oth if m != l] + [LD(1)]) for l in oth) / den
        return V, G

    V, G = basis(g)
    ends = basis(np.array([LD(0), LD(1)]))[1]
    return V.T @ (w[:, None] * V), G.T @ (w[:, None] * G), ends[0], ends[1]


def patch_matrices(k, sigma, ptype):
    """1-D SIPG stiffness and mass of the two-cell patch (h = 1); bit 0 / 1 of
    the type: left / right end on the domain boundary."""
    n = k + 1
    M, S, d0, d1 = cell_matrices(k)
    Z = np.zeros((n, n), LD)
    A, Mp = np.block([[S, Z], [Z, S]]), np.block([[M, Z], [Z, M]])
    for f in range(3):
        jump, mean = np.zeros(2 * n, LD), np.zeros(2 * n, LD)
        half = LD(1) if (f == 0 and ptype & 1) or (f == 2 and ptype & 2) else LD(0.5)
        if f > 0:
            jump[f * n - 1] += 1
            mean[(f - 1) * n:f * n] += half * d1
        if f < 2:
            jump[f * n] -= 1
            mean[f * n:(f + 1) * n] += half * d0
        A += sigma * np.outer(jump, jump) - np.outer(jump, mean) - np.outer(mean, jump)
    return A, Mp


@pytest.mark.parametrize("k", range(1, 8))
@pytest.mark.parametrize("ptype", [0, 1, 2])
@pytest.mark.parametrize("variant", [dgmg.SMOOTH_EXACT, dgmg.SMOOTH_FULL])
def test_eigenpairs_to_rounding(k, ptype, variant):
    sigma, E, u = inputs.sigma_of(k), 2 * (k + 1), 2.0 ** -53
    A, _ = patch_matrices(k, LD(sigma), ptype)
    S, lam = dgmg.patch_eigen(k, sigma, ptype, variant)
    used = np.isfinite(lam)
    S, lam = S[:, used].astype(LD), lam[used].astype(LD)
    R = np.abs(S.T @ A @ S - np.diag(lam)) / np.sqrt(np.outer(lam, lam))
    # A and S known to a round-off, two sums of E terms
    assert R.max() <= 4 * E * u
