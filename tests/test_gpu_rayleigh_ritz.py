"""The Rayleigh-Ritz step (Algorithm 3) at the sizes where its kernels change:
the padded sizes 4, 8, 10, 12, 16, 24 and their neighbours, the 16-column edge
of the thread grid, one column, and the structures that take other paths
(dropped and zero columns, exactly decoupled and clustered Ritz values).

Tolerances.  The step is a congruence with the Cholesky factor of the
unit-diagonal Gram matrix followed by an orthogonal eigensolver, both backward
stable: with at most 24 columns and a scaled Gram matrix of condition below
1e3 (checked), errors stay below 24^2 * 1e3 * 2^-53 ~ 6e-11 relative in the
worst case; Ritz values, B-orthonormality and the residual of the pencil are
gated at 1e-11."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 1e-11


def _check(gsf, GA, GB, m, drop_tol=1e-10, zero_tol=1e-13):
    th, C, kept, nk = gsf.rayleigh_ritz(GA, GB, m, drop_tol, zero_tol)
    rth, _, rkept = oracle.rayleigh_ritz(GA, GB, m, drop_tol, zero_tol)
    assert np.array_equal(kept, rkept) and nk == np.count_nonzero(rkept)
    d = np.sqrt(np.diag(GB)[kept])
    A, B = (G[np.ix_(kept, kept)] / d[:, None] / d for G in (GA, GB))
    assert np.linalg.cond(B) < 1e3
    Z = C[kept] * d[:, None]
    scale = np.linalg.norm(A, 2)
    assert np.abs(th - rth).max() <= TOL * scale
    assert np.all(np.diff(th) >= -TOL * scale)
    assert np.abs(Z.T @ B @ Z - np.eye(m)).max() <= TOL
    assert np.abs(A @ Z - B @ Z * th).max() <= TOL * scale
    assert not C[~kept].any()
    lead = C[np.abs(C).argmax(0), np.arange(m)]
    assert np.all(lead > 0.0)


@pytest.mark.parametrize("ns,m", [(1, 1), (2, 1), (3, 1), (4, 2), (5, 5), (8, 4), (9, 3), (10, 4), (11, 4), (12, 4),
                                  (13, 5), (15, 5), (16, 8), (17, 6), (21, 7), (23, 8), (24, 8), (24, 3)])
def test_sizes(gsf, ns, m):
    rng = np.random.default_rng(100 * ns + m)
    S = rng.standard_normal((300, ns)) * 10.0 ** rng.uniform(-6, 2, ns)
    lam = np.linspace(0.0, 1.0, 300) ** 3 * 2.0
    _check(gsf, S.T @ (lam[:, None] * S), S.T @ S, m)


@pytest.mark.parametrize("ns,m", [(6, 3), (12, 4), (16, 8), (24, 8)])
def test_decoupled_and_clustered(gsf, ns, m):
    rng = np.random.default_rng(ns)
    I = np.eye(ns)
    _check(gsf, np.diag(rng.uniform(0, 2, ns)), I, m)                 # no coupling at all
    _check(gsf, np.diag(np.repeat(0.5, ns)), I, m)                    # one eigenvalue
    Q, _ = np.linalg.qr(rng.standard_normal((ns, ns)))
    lam = np.sort(rng.uniform(0, 2, ns))
    lam[:m] = 1e-3 + 1e-14 * np.arange(m)                             # a cluster at rounding distance
    A = (Q * lam) @ Q.T
    _check(gsf, 0.5 * (A + A.T), I, m)
    lam[:m] = 1e-3 + 1e-8 * np.arange(m)                              # separated below 1e-7
    A = (Q * lam) @ Q.T
    _check(gsf, 0.5 * (A + A.T), I, m)


@pytest.mark.parametrize("ns,m,drop", [(6, 2, [3]), (12, 4, [0, 5, 11]), (17, 5, [16]), (24, 8, [8, 9, 15, 16, 23])])
def test_dropped_columns(gsf, ns, m, drop):
    rng = np.random.default_rng(7 * ns)
    S = rng.standard_normal((200, ns))
    lam = np.linspace(0.0, 1.5, 200)
    for k, j in enumerate(drop):
        S[:, j] = 0.0 if k % 2 == 0 else S[:, j - 1] * 3.0            # a zero column, a copy
    GA, GB = S.T @ (lam[:, None] * S), S.T @ S
    _check(gsf, GA, GB, m)
    # fewer columns than asked for
    G1 = np.ones((ns, ns))
    th, C, kept, nk = gsf.rayleigh_ritz(G1, G1, m, 1e-10, 1e-13)
    assert nk == 1 and kept[0] and not kept[1:].any()


@pytest.mark.parametrize("ns,m", [(3, 1), (4, 2), (9, 3), (12, 4), (16, 5), (24, 8)])
def test_small_ritz_values_of_a_diagonal_pencil(gsf, ns, m):
    """The bisection ends at 2^-60 of the Gershgorin interval (below 3 wide).  On
    a diagonal matrix the counts are exact, so a Ritz value is within half of
    that bracket, 1.3e-18, and the roundings of the bracket's ends, an ulp."""
    rng = np.random.default_rng(ns)
    for small in (1e-2, 1e-3, 1e-4):
        lam = np.concatenate([small * (1.0 + np.arange(m) + 0.3 * rng.uniform(size=m)), rng.uniform(0.5, 2.0, ns - m)])
        th = gsf.rayleigh_ritz(np.diag(lam), np.eye(ns), m, 1e-10, 1e-13)[0]
        ref = np.sort(lam)[:m]
        assert np.all(np.abs(th - ref) <= 1.3e-18 + 2 * np.spacing(ref))


@pytest.mark.parametrize("ns,m", [(6, 2), (9, 3), (12, 4), (17, 5), (24, 8)])
def test_columns_that_are_not_numbers(gsf, ns, m):
    """A column of NaN products is dropped and leaves the others as they are
    without it; so is the later one of two columns whose product alone is NaN."""
    rng = np.random.default_rng(3 * ns)
    S = rng.standard_normal((200, ns))
    lam = np.linspace(0.0, 1.5, 200)
    GA, GB = S.T @ (lam[:, None] * S), S.T @ S
    for j in (0, 3, ns - 1):
        rest = np.arange(ns) != j
        ref = oracle.rayleigh_ritz(GA[np.ix_(rest, rest)], GB[np.ix_(rest, rest)], m, 1e-10, 1e-13)[0]
        for what in ("column", "entry"):
            A, B = GA.copy(), GB.copy()
            if what == "column":
                A[j], A[:, j], B[j], B[:, j] = (np.nan,) * 4
            elif j > 0:
                B[j, 0] = B[0, j] = np.nan
            else:
                continue
            th, C, kept, nk = gsf.rayleigh_ritz(A, B, m, 1e-10, 1e-13)
            assert nk == ns - 1 and np.array_equal(kept.astype(bool), rest), (j, what)
            assert np.abs(th - ref).max() <= TOL * np.linalg.norm(GA, 2) and not C[j].any()
            assert np.isfinite(C).all()


@pytest.mark.parametrize("power", [-300, -100, -40, 30])
@pytest.mark.parametrize("ns,m", [(3, 1), (4, 2), (9, 3), (12, 4), (17, 5), (24, 8)])
def test_pencils_of_any_scale(gsf, ns, m, power):
    """GA 2^power: a graph whose weights are all tiny, or a pencil far above one;
    the gates are relative to the pencil's norm."""
    rng = np.random.default_rng(11 * ns + m)
    S = rng.standard_normal((200, ns))
    lam = np.linspace(0.0, 1.5, 200)
    GA, GB = S.T @ (lam[:, None] * S), S.T @ S
    _check(gsf, np.ldexp(GA, power), GB, m)


@pytest.mark.parametrize("coupling", [1e-70, 1e-90, 1e-140])
@pytest.mark.parametrize("ns,m", [(3, 1), (6, 2), (12, 4), (24, 8)])
def test_couplings_near_nothing(gsf, ns, m, coupling):
    """Columns coupled by a product far below rounding, but not by zero."""
    rng = np.random.default_rng(5 * ns)
    E = rng.standard_normal((ns, ns)) * coupling
    _check(gsf, np.diag(rng.uniform(0.1, 2.0, ns)) + 0.5 * (E + E.T), np.eye(ns), m)
