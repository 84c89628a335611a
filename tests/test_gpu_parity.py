"""GPU parity: every step of the HIP path, called through the C ABI, against
the FP64 CPU oracle on the same seeded inputs.

Tolerances (relative, 2-norm and max-norm over the whole output):
  FP64 path: 1e-12 for weights, apply and power iteration; the CG and LOBPCG
             outputs max(1e-12, 10 band), where the band is the oracle's own
             self-sensitivity (the same filter on the grid in reverse point
             order, which only reorders its sums; tests/sensitivity.py),
             measured for each case as it runs.
  FP32 path: 1e-5 for weights, apply, power iteration, CG and LOBPCG
             outputs; LOBPCG Ritz values within 1e-5 * ||L_sym||
             (||L_sym|| <= 2).
LOBPCG runs compare their decisions first: the number of trial columns the
Rayleigh-Ritz steps dropped must equal the oracle's wherever the oracle's
reversed run takes the same decisions (a drop on the rounding threshold is
not fixed by the method).  For FP32 runs the oracle receives the
FP32-rounded inputs, so the comparison measures the kernel's arithmetic, not
the rounding of its inputs.
"""
import numpy as np
import pytest

import oracle
from sensitivity import reference
from synth import WORKLOADS, make_signal, piecewise_constant_1d, scene_2d

pytestmark = pytest.mark.gpu


def rel(a, b):
    a = np.asarray(a, dtype=np.float64).ravel()
    b = np.asarray(b, dtype=np.float64).ravel()
    den2 = max(np.linalg.norm(b), 1e-300)
    deni = max(np.abs(b).max(), 1e-300)
    return max(np.linalg.norm(a - b) / den2, np.abs(a - b).max() / deni)


def _inputs(case):
    """(shape, float64 noisy signal) of a named test case."""
    kind, shape, seed = case
    if len(shape) == 1:
        return shape, piecewise_constant_1d(shape[0], 0.1, seed)[1]
    return shape, scene_2d(shape[0], shape[1], 0.05, seed)[1]


def _torch(x, prec, gsf):
    import torch
    dt = torch.float32 if prec == gsf.F32 else torch.float64
    return torch.tensor(np.ascontiguousarray(x), dtype=dt, device="cuda")


def _round(x, prec, gsf):
    return x.astype(np.float32).astype(np.float64) if prec == gsf.F32 else x


TOL = {0: 1e-5, 1: 1e-12}

# (kind, shape, seed): sizes span several tiles plus ragged tails
BF_CASES = [("bf", (4096,), 1), ("bf", (1000,), 2), ("bf", (67, 130), 3), ("bf", (33, 200), 4)]
GF_CASES = [("gf", (1500,), 5), ("gf", (70, 131), 6)]

# operator parameters per case: 1D the 4096-sample signal's BF (radius 5,
# sigma_d 3, sigma_r 0.2); 67 x 130 the 1024^2 image's 11 x 11 window (radius
# 5, sigma_d 2, sigma_r 0.1); 33 x 200 a 7 x 7 window; GF radius 4 (1D) or 3
PARAMS = {
    (4096,): dict(radius=5, sigma_d=3.0, sigma_r=0.2),
    (1000,): dict(radius=5, sigma_d=3.0, sigma_r=0.2),
    (67, 130): dict(radius=5, sigma_d=2.0, sigma_r=0.1),
    (33, 200): dict(radius=3, sigma_d=2.0, sigma_r=0.1),
}


def _params(kind, shape):
    if kind == "bf":
        return dict(PARAMS[tuple(shape)])
    return dict(radius=4 if len(shape) == 1 else 3, eps=1e-2)


def _oracle_op(kind, grid, p):
    return oracle.build_operator(kind, grid, p["radius"], p.get("sigma_d", 0.0), p.get("sigma_r", 0.0),
                                 p.get("eps", 0.0))


def _build(gsf, case, prec):
    shape, x = _inputs(case)
    kind = case[0]
    p = _params(kind, shape)
    xr = _round(x, prec, gsf)
    op = gsf.Operator(kind, shape, _torch(x, prec, gsf), prec=prec, **p)
    ref = _oracle_op(kind, xr.reshape(shape), p)
    return op, ref, xr.ravel()


# ------------------------------------------------------------------ build
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", BF_CASES)
def test_bf_build_parity(gsf, case, prec):
    """Half-window planes against the oracle's W (w_{i,i+o}, 0 off the grid),
    degrees as the FP64 row sums of exactly the stored weights (own planes
    plus the mirrored entries w_{i-o,i}: D 1 = W 1 for the operator that is
    applied) and against the oracle's d, sqrt(d) and 1/sqrt(d).  FP32 data:
    the weights come from the FP32 exponential of the one-pass build, within
    a few units of 2^-24 times 1 + the exponent's magnitude of the oracle's."""
    op, ref, _ = _build(gsf, case, prec)
    planes = op.planes().cpu().numpy().astype(np.float64)
    shape = ref.shape
    r = ref.radius
    W = ref.W.tocsr()
    n = ref.n
    offs = [(o,) for o in range(1, r + 1)] if len(shape) == 1 else \
        [(0, dx) for dx in range(1, r + 1)] + [(dy, dx) for dy in range(1, r + 1) for dx in range(-r, r + 1)]
    assert planes.shape[0] == len(offs)
    coords = np.indices(shape).reshape(len(shape), -1).T
    d_st = np.ones(n)
    for q, o in enumerate(offs):
        nb = coords + np.array(o)
        inside = np.all((nb >= 0) & (nb < np.array(shape)), axis=1)
        i = np.flatnonzero(inside)
        j = np.ravel_multi_index(tuple(nb[inside].T), shape)
        expect = np.zeros(n)
        expect[i] = np.asarray(W[i, j]).ravel()
        assert rel(planes[q], expect) <= TOL[prec], (q, o)
        assert np.all(planes[q][~inside] == 0.0)
        d_st[i] += planes[q][i]   # own half: w_{i,i+o}
        d_st[j] += planes[q][i]   # mirrored half: w_{j-o,j} = w_{i,i+o} at j = i + o
    deg = op.degree().cpu().numpy()
    np.testing.assert_allclose(deg, d_st, rtol=1e-13)
    assert rel(deg, ref.d) <= (1e-13 if prec == gsf.F64 else TOL[prec])
    assert rel(op.sqrt_d().cpu().numpy(), ref.sqrt_d) <= TOL[prec]
    assert rel(op.inv_sqrt_d().cpu().numpy(), 1.0 / ref.sqrt_d) <= TOL[prec]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", GF_CASES)
def test_gf_build_parity(gsf, case, prec):
    op, ref, _ = _build(gsf, case, prec)
    mu, inv = op.gf_stats()
    rmu, rinv = ref.gf_window_stats()
    assert rel(mu.cpu().numpy(), rmu) <= TOL[prec]
    assert rel(inv.cpu().numpy(), rinv) <= (TOL[prec] if prec == 1 else 1e-5)
    np.testing.assert_allclose(op.degree().cpu().numpy(), ref.d, rtol=1e-15)


# ------------------------------------------------------------------ apply
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m", [1, 3, 4, 8])
@pytest.mark.parametrize("case", BF_CASES[1:] + GF_CASES)
def test_apply_parity_all_forms(gsf, case, prec, m):
    op, ref, _ = _build(gsf, case, prec)
    rng = np.random.default_rng(100 + m)
    X = _round(rng.standard_normal((op.n, m)), prec, gsf)
    Xd = _torch(X if m > 1 else X[:, 0], prec, gsf)
    for form in (gsf.FORM_N, gsf.FORM_LSYM, gsf.FORM_RW):
        Y = op.apply(Xd, form).cpu().numpy().reshape(op.n, m)
        R = ref.apply(form, X)
        assert rel(Y, R) <= TOL[prec], (form, rel(Y, R))


def test_apply_deterministic(gsf):
    op, ref, x = _build(gsf, ("bf", (67, 130), 3), 0)
    xd = _torch(x, 0, gsf)
    a = op.apply(xd, gsf.FORM_LSYM).cpu().numpy()
    b = op.apply(xd, gsf.FORM_LSYM).cpu().numpy()
    assert np.array_equal(a, b)


# ------------------------------------------------------------------ power iteration
@pytest.mark.parametrize("prec,case,k", [(1, ("bf", (4096,), 1), 30), (0, ("bf", (67, 130), 3), 20),
                                         (1, ("gf", (70, 131), 6), 10), (0, ("gf", (1500,), 5), 10)])
def test_power_filter_parity(gsf, prec, case, k):
    op, ref, x = _build(gsf, case, prec)
    y = op.power_filter(_torch(x, prec, gsf), k).cpu().numpy()
    r = oracle.power_filter(ref, x, k)
    err = rel(y, r)
    print(f"power {case} prec={prec} k={k}: rel err {err:.3e}")
    assert err <= TOL[prec], err


# ------------------------------------------------------------------ CG
def _grid(x, shape):
    return np.asarray(x, dtype=np.float64).reshape(shape)


@pytest.mark.parametrize("prec,case,k", [(1, ("bf", (4096,), 1), 30), (1, ("bf", (67, 130), 3), 30),
                                         (0, ("bf", (67, 130), 3), 30), (1, ("gf", (70, 131), 6), 20),
                                         (0, ("bf", (33, 200), 4), 50), (1, ("bf", (33, 200), 4), 50)])
def test_cg_filter_parity(gsf, prec, case, k):
    op, _, x = _build(gsf, case, prec)
    p = _params(case[0], op.shape)
    dp = "f32" if prec == 0 else "f64"
    y, info = op.cg_filter(_torch(x, prec, gsf), k)
    ref = reference(lambda g: oracle.cg_filter(_oracle_op(case[0], g, p), g.ravel(), k, data_prec=dp),
                    _grid(x, op.shape))
    rinfo = ref.extra
    assert info.iters == rinfo.iters and info.status == 0
    err = rel(y.cpu().numpy(), ref.y)
    gate = ref.gate if prec == 1 else TOL[0]
    print(f"cg {case} prec={prec} k={k}: rel err {err:.3e} (band {ref.band:.1e}, gate {gate:.1e})")
    assert err <= gate, err
    assert abs(info.res0 - rinfo.res0) <= 1e-6 * rinfo.res0


def test_cg_constant_input_breakdown(gsf):
    import torch
    shape = (40, 70)
    x = np.full(shape, 0.3)
    op = gsf.Operator("bf", shape, _torch(x, 1, gsf), radius=2, sigma_d=2.0, sigma_r=0.1, prec=gsf.F64)
    y, info = op.cg_filter(_torch(x.ravel(), 1, gsf), 10)
    assert info.status == gsf.EBREAKDOWN and info.iters == 0
    np.testing.assert_array_equal(y.cpu().numpy(), x.ravel())


def test_cg_tolerance_stop(gsf):
    op, _, x = _build(gsf, ("bf", (1000,), 2), 1)
    p = _params("bf", op.shape)
    y, info = op.cg_filter(_torch(x, 1, gsf), 500, tol=1e-6)
    ref = reference(lambda g: oracle.cg_filter_normalized(_oracle_op("bf", g, p), g, 500, tol=1e-6), x)
    assert ref.extra.iters == ref.extra_reversed.iters
    assert info.status == 0 and info.iters == ref.extra.iters
    assert rel(y.cpu().numpy(), ref.y) <= ref.gate


# ------------------------------------------------------------------ Gram (MFMA) and Rayleigh-Ritz
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m,nb", [(1, 1), (3, 3), (4, 3), (5, 3), (8, 2), (8, 3)])
def test_block_gram_parity(gsf, prec, m, nb):
    import torch
    n = 5003
    rng = np.random.default_rng(7 + m + nb)
    S = [_round(rng.standard_normal((n, m)), prec, gsf) for _ in range(nb)]
    A = [_round(rng.standard_normal((n, m)), prec, gsf) for _ in range(nb)]
    GA, GB = gsf.block_gram([_torch(s, prec, gsf) for s in S], [_torch(a, prec, gsf) for a in A], prec=prec)
    Sf, Af = np.column_stack(S), np.column_stack(A)
    assert rel(GB, Sf.T @ Sf) <= 1e-13
    assert rel(GA, Sf.T @ Af) <= 1e-13
    # entry by entry: products of FP32 or FP64 data summed in FP64 stay within
    # the textbook bound n 2^-53 |S|^T |A| of the exact sum (FP32 sums would
    # not, on entries much smaller than their terms)
    bound = n * 2.0 ** -53
    assert np.all(np.abs(GB - Sf.T @ Sf) <= bound * (np.abs(Sf).T @ np.abs(Sf)))
    assert np.all(np.abs(GA - Sf.T @ Af) <= bound * (np.abs(Sf).T @ np.abs(Af)))


@pytest.mark.parametrize("ns,m,drop", [(1, 1, False), (2, 1, False), (9, 3, False), (16, 4, False),
                                       (17, 5, False), (23, 8, False), (24, 8, False), (12, 4, True),
                                       (24, 8, True)])
def test_rayleigh_ritz_parity(gsf, ns, m, drop):
    """The single-wave Rayleigh-Ritz step against the oracle's: even and odd
    kept counts (a dummy player in the Jacobi schedule), up to 24 columns
    (more 2 x 2 blocks than lanes), with nearly dependent columns dropped."""
    rng = np.random.default_rng(ns)
    S = rng.standard_normal((200, ns))
    if drop:
        S[:, 7] = 2.0 * S[:, 2] + 1e-9 * rng.standard_normal(200)
        if ns > 20:
            S[:, 19] = S[:, 3] - S[:, 11] + 1e-9 * rng.standard_normal(200)
    A0 = rng.standard_normal((200, 200))
    A = A0 @ A0.T / 200
    GA, GB = S.T @ A @ S, S.T @ S
    th, C, kept, nk = gsf.rayleigh_ritz(GA, GB, m, 1e-10, 1e-13)
    rth, rC, rkept = oracle.rayleigh_ritz(GA, GB, m, 1e-10, 1e-13)
    assert np.array_equal(kept, rkept)
    np.testing.assert_allclose(th, rth, rtol=1e-11, atol=1e-12)
    # columns agree up to sign
    for j in range(m):
        sgn = np.sign(C[:, j] @ rC[:, j])
        assert rel(sgn * C[:, j], rC[:, j]) <= 1e-8


# ------------------------------------------------------------------ LOBPCG
def lobpcg_reference(kind, p, x, shape, m, k, prec, **kw):
    """The oracle's LOBPCG output with its band (FP64 data) and decisions."""
    dp = "f64" if prec == 1 else "f32"

    def run(g):
        y, th, X, info = oracle.lobpcg_filter(_oracle_op(kind, g, p), g.ravel(), m, k, data_prec=dp, **kw)
        return y, (th, info)

    return reference(run, _grid(x, shape))


def check_lobpcg(info, y, ref, m, prec, label=""):
    """Decisions first (steps; dropped columns where the oracle's reversed
    run agrees with itself), then Ritz values and the output."""
    th, rinfo = ref.extra
    _, rinfo_rev = ref.extra_reversed
    assert info.iters == rinfo.iters
    if rinfo.dropped == rinfo_rev.dropped:
        assert info.dropped == rinfo.dropped, (info.dropped, rinfo.dropped)
    theta = np.array(info.theta[:m])
    e = rel(y, ref.y)
    print(f"lobpcg {label} prec={prec}: y rel {e:.2e} (band {ref.band:.1e}), theta abs "
          f"{np.abs(theta - th).max():.2e}, dropped {info.dropped} vs {rinfo.dropped} "
          f"(reversed oracle {rinfo_rev.dropped})")
    if prec == 1:
        np.testing.assert_allclose(theta, th, rtol=max(1e-9, ref.gate), atol=1e-12)
        assert e <= ref.gate, e
    else:
        assert np.abs(theta - th).max() <= 2e-5
        assert e <= TOL[0], e
    return e


@pytest.mark.parametrize("prec,case,m,k,constraint", [
    (1, ("bf", (4096,), 1), 3, 30, False),
    (1, ("bf", (4096,), 1), 3, 30, True),
    (1, ("bf", (67, 130), 3), 4, 20, False),
    (1, ("gf", (70, 131), 6), 4, 10, True),
    (0, ("bf", (67, 130), 3), 4, 20, True),
    (0, ("bf", (33, 200), 4), 8, 15, False),
    (1, ("bf", (33, 200), 4), 8, 15, True),   # widest block with the constraint: m + 1 output coefficients
])
def test_lobpcg_filter_parity(gsf, prec, case, m, k, constraint):
    import torch
    op, _, x = _build(gsf, case, prec)
    p = _params(case[0], op.shape)
    ritz = torch.empty((op.n, m), dtype=op.dtype, device="cuda")
    y, info = op.lobpcg_filter(_torch(x, prec, gsf), m, k, constraint=constraint, ritz=ritz)
    ref = lobpcg_reference(case[0], p, x, op.shape, m, k, prec, constraint=constraint)
    check_lobpcg(info, y.cpu().numpy(), ref, m, prec, f"{case} m={m} k={k} c={constraint}")


@pytest.mark.parametrize("prec,m", [(0, 1), (0, 2), (1, 1)])
@pytest.mark.parametrize("shape", [(23, 45), (46, 29), (25, 41), (33, 31)])
@pytest.mark.parametrize("constraint", [False, True])
def test_lobpcg_narrow_block_groups(gsf, shape, prec, m, constraint):
    """LOBPCG with rows of less than 16 bytes, whose update takes several points
    at a time: every remainder of the point count, all three basis widths
    (first, second and later steps), and the projection of narrow rows."""
    x = _round(scene_2d(*shape, 0.05, 9)[1], prec, gsf)
    p = dict(radius=2, sigma_d=2.0, sigma_r=0.2)
    op = gsf.Operator("bf", shape, _torch(x.ravel(), prec, gsf), prec=prec, **p)
    y, info = op.lobpcg_filter(_torch(x.ravel(), prec, gsf), m, 6, constraint=constraint)
    ref = lobpcg_reference("bf", p, x, shape, m, 6, prec, constraint=constraint)
    check_lobpcg(info, y.cpu().numpy(), ref, m, prec, f"{shape} m={m} c={constraint}")


def test_lobpcg_identity_at_zero_steps(gsf):
    op, ref, x = _build(gsf, ("bf", (67, 130), 3), 1)
    y, info = op.lobpcg_filter(_torch(x, 1, gsf), 4, 0)
    assert rel(y.cpu().numpy(), x) <= 1e-12


def test_lobpcg_constant_input_breakdown(gsf):
    shape = (30, 64)
    x = np.full(shape, 0.3)
    op = gsf.Operator("bf", shape, _torch(x, 1, gsf), radius=2, sigma_d=2.0, sigma_r=0.1, prec=gsf.F64)
    y, info = op.lobpcg_filter(_torch(x.ravel(), 1, gsf), 2, 5, constraint=True)
    assert info.status == gsf.EBREAKDOWN
    np.testing.assert_array_equal(y.cpu().numpy(), x.ravel())


# ------------------------------------------------------------------ precision study
@pytest.mark.parametrize("kind", ["bf7", "gf8"])
@pytest.mark.parametrize("prec", [0, 1])
def test_precision_study_lobpcg_m8_100_steps(gsf, kind, prec):
    """The precision-study configuration (noise 0.08; BF 7x7 with sigma_d = 2,
    sigma_r = 0.15, or GF radius 8 with eps = 1e-2; LOBPCG m = 8, 100 steps)
    at a size the oracle finishes in seconds.  FP64: Ritz values and output
    within the band gate (100 steps of an m = 8 block amplify
    summation-order differences: the BF band is ~5e-12).  FP32 (FP32 data and
    MFMA Gram, FP64 Rayleigh-Ritz): Ritz values within 1e-5 * ||L_sym||
    (||L_sym|| <= 2); the output error is reported, as the precision study
    reports it: y projects z0 on all eight Ritz vectors, the upper ones far
    from converged after 100 steps, and FP32 rounding moves their span and
    the drop decisions (measured: BF 7x7 8.7e-4 with 90 drops against the
    oracle's 106, Ritz values within 4.4e-9).  The GF run converges its first
    column to the null vector within a few steps; its trial columns then sit
    at the rounding level and are dropped on rounding decisions that the
    oracle itself takes differently when its sums are reordered, so the drop
    counts are compared only where the oracle agrees with itself."""
    H, W = 96, 112
    x = scene_2d(H, W, 0.08, 3)[1]
    xr = _round(x, prec, gsf)
    p = dict(radius=3, sigma_d=2.0, sigma_r=0.15) if kind == "bf7" else dict(radius=8, eps=1e-2)
    okind = "bf" if kind == "bf7" else "gf"
    op = gsf.Operator(okind, (H, W), _torch(xr, prec, gsf), prec=prec, **p)
    m, k = 8, 100
    y, info = op.lobpcg_filter(_torch(xr, prec, gsf), m, k)
    ref = lobpcg_reference(okind, p, xr, (H, W), m, k, prec)
    th, rinfo = ref.extra
    theta = np.array(info.theta[:m])
    ey = rel(y.cpu().numpy(), ref.y)
    et = np.abs(theta - th).max()
    print(f"precision study {kind} prec {prec}: theta abs {et:.2e} (rel {np.abs(theta / th - 1).max():.2e}), "
          f"y rel {ey:.2e} (band {ref.band:.1e}), dropped {info.dropped} vs {rinfo.dropped} "
          f"(reversed oracle {ref.extra_reversed[1].dropped})")
    assert info.iters == rinfo.iters == k
    if prec == 1:
        check_lobpcg(info, y.cpu().numpy(), ref, m, prec, f"precision study {kind}")
    else:
        assert et <= 2e-5


# ------------------------------------------------------------------ the 1024^2 image's operator at 256^2
@pytest.fixture(scope="module")
def crop256():
    """The top-left 256 x 256 crop of the 1024^2 workload image (noise 0.05,
    seed 2) with its operator parameters (BF 11 x 11, sigma_d 2, sigma_r 0.1)."""
    w = WORKLOADS["image_1024_bf11"]
    x = make_signal("image_1024_bf11")[1][:256, :256].copy()
    return x, dict(radius=w["radius"], sigma_d=w["sigma_d"], sigma_r=w["sigma_r"])


@pytest.mark.parametrize("prec", [0, 1])
def test_image_crop_cg50_lobpcg_m4_50_and_joint(gsf, crop256, prec):
    """The bench step's filters on a 256^2 crop of its image, element by
    element against the oracle: CG 50 steps, LOBPCG m = 4 50 steps (the 11 x 11
    stored-plane apply, the MFMA Gram and the FP64 Rayleigh-Ritz step) and the
    joint driver, whose shared stencil pass is the bench's timed kernel."""
    x, p = crop256
    xr = _round(x, prec, gsf)
    shape = xr.shape
    op = gsf.Operator("bf", shape, _torch(xr.ravel(), prec, gsf), prec=prec, **p)
    xd = _torch(xr.ravel(), prec, gsf)
    dp = "f32" if prec == 0 else "f64"
    rcg = reference(lambda g: oracle.cg_filter(_oracle_op("bf", g, p), g.ravel(), 50, data_prec=dp), xr)
    rlob = lobpcg_reference("bf", p, xr, shape, 4, 50, prec)
    cg_gate = rcg.gate if prec == 1 else TOL[0]
    y, info = op.cg_filter(xd, 50)
    e = rel(y.cpu().numpy(), rcg.y)
    print(f"crop CG 50 prec {prec}: {e:.2e} (band {rcg.band:.1e})")
    assert info.iters == rcg.extra.iters == 50 and e <= cg_gate
    y, info = op.lobpcg_filter(xd, 4, 50)
    check_lobpcg(info, y.cpu().numpy(), rlob, 4, prec, "crop m=4 k=50")
    for rows in (None, 1, 2, 4):
        if rows is not None:
            op.set_apply_rows(4, rows)
        ycg, ylob, ci, li = op.joint_filter(xd, 50, xd, 4, 50)
        e = rel(ycg.cpu().numpy(), rcg.y)
        print(f"crop joint rows={rows} prec {prec}: cg {e:.2e}")
        assert ci.iters == 50 and e <= cg_gate
        check_lobpcg(li, ylob.cpu().numpy(), rlob, 4, prec, f"crop joint rows={rows}")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [777, 8192, 8193, 12000])
def test_cg_1d_small_and_large_paths(gsf, n, prec):
    """1D BF CG: up to 8192 samples the filter runs in one workgroup, above on
    the multi-kernel path; both against the oracle, with a tolerance stop at
    the oracle's step and a breakdown for a constant input."""
    x = piecewise_constant_1d(n, 0.1, 40 + n)[1]
    xr = _round(x, prec, gsf)
    op = gsf.Operator("bf", (n,), _torch(xr, prec, gsf), radius=4, sigma_d=3.0, sigma_r=0.2, prec=prec)
    ref = oracle.build_operator("bf", xr, 4, 3.0, 0.2)
    dp = "f32" if prec == 0 else "f64"
    y, info = op.cg_filter(_torch(xr, prec, gsf), 25)
    rr = reference(lambda g: oracle.cg_filter(oracle.build_operator("bf", g, 4, 3.0, 0.2), g, 25, data_prec=dp), xr)
    r, rinfo = rr.y, rr.extra
    e = rel(y.cpu().numpy(), r)
    print(f"cg 1D n={n} prec={prec}: {e:.2e} (band {rr.band:.1e})")
    assert info.iters == rinfo.iters == 25 and info.status == gsf.OK and e <= (rr.gate if prec else TOL[0])
    assert abs(info.res0 - rinfo.res0) <= 1e-6 * rinfo.res0
    y, info = op.cg_filter(_torch(xr, prec, gsf), 2000, tol=1e-4)
    r, rinfo = oracle.cg_filter(ref, xr, 2000, tol=1e-4, data_prec=dp)
    assert info.status == gsf.OK and abs(info.iters - rinfo.iters) <= (0 if prec else 2)
    c = np.full(n, 0.4)
    y, info = op.cg_filter(_torch(c, prec, gsf), 10)
    assert info.status == gsf.EBREAKDOWN and info.iters == 0
    np.testing.assert_allclose(y.cpu().numpy(), c, rtol=1e-6 if prec == 0 else 1e-15)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("radius", [1, 2, 3, 5, 6, 8])
@pytest.mark.parametrize("n", [2, 63, 65, 1024, 1025, 2048, 2049, 4096, 4097, 8191])
def test_cg_1d_one_workgroup_forms(gsf, n, radius, prec):
    """The one-workgroup CG where its forms meet: one wave or less, the lengths
    at which a thread takes one, two, four or eight points, radii whose weights
    stay in registers and radii whose do not, windows wider than the signal;
    the same steps as the oracle, twice the same bits."""
    import torch
    x = _round(piecewise_constant_1d(n, 0.1, 11)[1] if n > 2 else np.array([0.2, 0.7]), prec, gsf)
    op = gsf.Operator("bf", (n,), _torch(x, prec, gsf), radius=radius, sigma_d=3.0, sigma_r=0.2, prec=prec)
    dp = "f32" if prec == 0 else "f64"
    kmax = 1 if n == 2 else 8
    rr = reference(lambda g: oracle.cg_filter(oracle.build_operator("bf", g, radius, 3.0, 0.2), g, kmax, data_prec=dp),
                   x)
    y, info = op.cg_filter(_torch(x, prec, gsf), kmax)
    e = rel(y.cpu().numpy(), rr.y)
    assert info.iters == rr.extra.iters == kmax
    assert e <= (rr.gate if prec else TOL[0]), e
    assert torch.equal(op.cg_filter(_torch(x, prec, gsf), kmax)[0], y)


@pytest.mark.parametrize("offset", [0, 8])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(3, 5), (1, 1023), (64, 64), (91, 90), (725, 725)])
def test_cg_step_chunks(gsf, shape, prec, offset):
    """The CG step's vector phases in 16-byte chunks: fewer points than a chunk
    row, every remainder, several chunks per thread (above 524288 points in
    FP32); and a workspace off the 16-byte grid, where they take elements."""
    import torch
    x = _round(scene_2d(*shape, 0.05, 5)[1] if min(shape) > 1 else
               np.random.default_rng(5).uniform(0, 1, shape), prec, gsf)
    xd = _torch(x.ravel(), prec, gsf)
    op = gsf.Operator("bf", shape, xd, radius=1, sigma_d=2.0, sigma_r=0.2, prec=prec)
    need = op.workspace(gsf.METHOD_CG).numel()
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")[offset:offset + need]
    dp = "f32" if prec == 0 else "f64"
    rr = reference(lambda g: oracle.cg_filter(oracle.build_operator("bf", g.reshape(shape), 1, 2.0, 0.2), g, 8,
                                              data_prec=dp), x.ravel())
    y, info = op.cg_filter(xd, 8, ws=ws)
    e = rel(y.cpu().numpy(), rr.y)
    print(f"cg chunks {shape} prec={prec} offset={offset}: {e:.2e}")
    assert info.status == gsf.OK and info.iters == 8
    assert e <= (rr.gate if prec else TOL[0])


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,radius", [((5, 9), 3), ((9, 5), 3), ((1, 700), 2), ((300, 1), 4), ((37, 500), 8),
                                          ((70, 131), 1), ((600,), 8), ((3,), 8), ((1,), 2)])
def test_gf_one_column_all_forms_edges(gsf, shape, radius, prec):
    """The GF apply of one column (FP32: the one-pass kernel; FP64: the two
    passes) on grids smaller than the window, single rows and columns, several
    256-column strips, tiny 1D signals, every radius class; all four forms,
    a strided x / y (every third point of a wider array) against the oracle."""
    import torch
    rng = np.random.default_rng(7 + radius)
    g = rng.uniform(0.0, 1.0, shape)
    g = _round(g, prec, gsf)
    op = gsf.Operator("gf", shape, _torch(g.ravel(), prec, gsf), radius=radius, eps=1e-2, prec=prec)
    ref = oracle.build_operator("gf", g, radius, eps=1e-2)
    x = _round(rng.standard_normal(op.n), prec, gsf)
    wide = np.zeros((op.n, 3))
    wide[:, 1] = x
    xd = _torch(wide, prec, gsf)
    for form in (gsf.FORM_N, gsf.FORM_LSYM, gsf.FORM_RW, gsf.FORM_L):
        y = op.apply(xd[:, 1:2], form).cpu().numpy().ravel()
        yw = torch.zeros_like(xd)
        op.apply(xd[:, 1:2], form, out=yw[:, 2:3])
        r = ref.apply(form, x)
        # relative to the input's scale: a Laplacian form can vanish (one point)
        scale = max(np.linalg.norm(r), np.linalg.norm(x))
        e = max(np.linalg.norm(y - r) / scale, np.abs(y - r).max() / max(np.abs(r).max(), np.abs(x).max()))
        assert e <= TOL[prec], (form, e)
        assert np.array_equal(yw[:, 2].cpu().numpy(), y)
        assert not yw[:, 0].any() and not yw[:, 1].any()


@pytest.mark.parametrize("radius", [1, 3, 6, 8])
@pytest.mark.parametrize("shape", [(3, 4), (9, 7), (40, 223), (33, 224), (21, 225), (17, 226), (50, 240), (8, 449),
                                   (130, 500), (1030, 12), (700,), (1793,)])
def test_gf_one_column_strips(gsf, shape, radius):
    """The one-pass GF apply on contiguous columns where its strips and chunks
    begin and end: widths of one strip's outputs and one column more or less,
    every remainder by the four columns of a lane, strips off the grid on one
    or both sides, odd chunk heights, rows too few for the straight-line part;
    all four forms, and the CG filter (whose p^T q the apply sums), against the
    oracle, and against the element-by-element form (strided columns)."""
    import torch
    rng = np.random.default_rng(70 + radius)
    g = _round(rng.uniform(0.0, 1.0, shape), gsf.F32, gsf)
    op = gsf.Operator("gf", shape, _torch(g.ravel(), gsf.F32, gsf), radius=radius, eps=1e-2, prec=gsf.F32)
    ref = oracle.build_operator("gf", g, radius, eps=1e-2)
    x = _round(rng.standard_normal(op.n), gsf.F32, gsf)
    xd = _torch(x, gsf.F32, gsf)
    wide = torch.zeros((op.n, 2), device="cuda")
    wide[:, 0] = xd
    for form in (gsf.FORM_N, gsf.FORM_LSYM, gsf.FORM_RW, gsf.FORM_L):
        y = op.apply(xd.reshape(-1, 1), form).ravel()
        assert torch.equal(op.apply(wide[:, 0:1], form).ravel(), y)
        r = ref.apply(form, x)
        e = np.linalg.norm(y.cpu().numpy() - r) / max(np.linalg.norm(r), np.linalg.norm(x))
        assert e <= TOL[gsf.F32], (form, e)
    y, info = op.cg_filter(_torch(g.ravel(), gsf.F32, gsf), 5)
    r, rinfo = oracle.cg_filter(ref, g.ravel(), 5, data_prec="f32")
    e = rel(y.cpu().numpy(), r)
    assert info.iters == rinfo.iters and e <= TOL[gsf.F32], e


@pytest.mark.parametrize("shape,radius", [((41, 700), 8), ((41, 699), 8), ((30, 480), 1), ((900,), 5)])
def test_gf_one_column_reach_of_a_value(gsf, shape, radius):
    """The one-pass GF apply takes its horizontal sums from prefix sums of 64
    columns: a pixel in column c enters the centres from c - r to r + 1 past the
    end of its piece, these the outputs to r + 1 past the end of the next piece.
    Every output left of c - 2r or right of c + 128 + r is the one of the clean
    image, to the bit: a large value first (it would take digits off the sums
    to its right), then ones that are not finite."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    n, cols = int(np.prod(shape)), shape[-1]
    g = torch.rand(n, device="cuda", generator=gen)
    x = torch.rand(n, device="cuda", generator=gen)
    op = gsf.Operator("gf", shape, g, radius=radius, eps=1e-2, prec=gsf.F32)
    clean = op.apply(x.reshape(-1, 1), gsf.FORM_N).reshape(-1, cols)
    row = (n // cols) // 2
    for c in (0, 20, 63, 64, 200, 230, cols - 1):
        for v in (1e30, float("inf"), float("nan")):
            bad = x.clone()
            bad[row * cols + c] = v
            y = op.apply(bad.reshape(-1, 1), gsf.FORM_N).reshape(-1, cols)
            lo, hi = max(c - 2 * radius, 0), c + 128 + radius + 1
            assert torch.equal(y[:, :lo], clean[:, :lo]), (c, v)
            assert torch.equal(y[:, hi:], clean[:, hi:]), (c, v)


@pytest.mark.parametrize("shape,radius", [((229376,), 8), ((229377,), 8), ((262144, 3), 1), ((262400, 3), 1)])
def test_gf_one_column_dot_by_apply_or_launch(gsf, shape, radius):
    """CG on the FP32 GF operator on both sides of 1024 apply workgroups: up to
    there the apply sums p^T q, above it a dot launch does."""
    rng = np.random.default_rng(31)
    g = _round(rng.uniform(0.0, 1.0, shape), gsf.F32, gsf)
    op = gsf.Operator("gf", shape, _torch(g.ravel(), gsf.F32, gsf), radius=radius, eps=1e-2, prec=gsf.F32)
    ref = oracle.build_operator("gf", g, radius, eps=1e-2)
    y, info = op.cg_filter(_torch(g.ravel(), gsf.F32, gsf), 5)
    r, rinfo = oracle.cg_filter(ref, g.ravel(), 5, data_prec="f32")
    e = rel(y.cpu().numpy(), r)
    assert info.iters == rinfo.iters and e <= TOL[gsf.F32], e


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m", [4, 8])
@pytest.mark.parametrize("shape,radius", [((3, 2), 8), ((9, 239), 8), ((40, 240), 8), ((33, 241), 3), ((70, 255), 1),
                                          ((21, 513), 6), ((2100, 64), 2), ((66000,), 5), ((500,), 8), ((1, 300), 4)])
def test_gf_block_strips(gsf, shape, radius, m, prec):
    """The GF apply of a block of 4 or 8 columns where its strips and chunks
    begin and end: a strip's 256 - 2r output columns and one more or less, a
    grid smaller than the window, several strips, tall narrow images and
    signals on both sides of the choice of kernel; all four forms against the
    oracle, and bit for bit against columns of a wider array."""
    import torch
    rng = np.random.default_rng(90 + radius)
    g = _round(rng.uniform(0.0, 1.0, shape), prec, gsf)
    op = gsf.Operator("gf", shape, _torch(g.ravel(), prec, gsf), radius=radius, eps=1e-2, prec=prec)
    ref = oracle.build_operator("gf", g, radius, eps=1e-2)
    x = _round(rng.standard_normal((op.n, m)), prec, gsf)
    xd = _torch(x, prec, gsf)
    wide = torch.zeros((op.n, m + 3), dtype=xd.dtype, device="cuda")
    wide[:, 1:1 + m] = xd
    for form in (gsf.FORM_N, gsf.FORM_LSYM, gsf.FORM_RW, gsf.FORM_L):
        y = op.apply(xd, form)
        out = torch.zeros_like(wide)
        op.apply(wide[:, 1:1 + m], form, out=out[:, 2:2 + m])
        assert torch.equal(out[:, 2:2 + m], y)
        assert not out[:, :2].any() and not out[:, 2 + m:].any()
        y = y.cpu().numpy()
        for j in (0, m - 1):
            r = ref.apply(form, x[:, j])
            e = np.linalg.norm(y[:, j] - r) / max(np.linalg.norm(r), np.linalg.norm(x[:, j]))
            assert e <= TOL[prec], (form, j, e)


@pytest.mark.parametrize("prec,m", [(0, 4), (0, 8), (1, 4), (1, 8)])
@pytest.mark.parametrize("shape,radius", [((2500, 2300), 8), ((9000, 64), 8), ((40000, 240), 1)])
def test_gf_block_rows_start_afresh(gsf, shape, radius, m, prec):
    """The running window sums of a block's apply start afresh at least every
    32 rows, whatever the image's height: what a row holds reaches (beside the
    window's r rows, in each of the two passes) the 31 rows after it at most.
    Exact: a perturbed row 0 leaves every output from row 2 (31 + r) + 1 on as
    it was, to the bit; a large value first (it would take digits off the sums
    below it), then a NaN."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3)
    dt = torch.float32 if prec == gsf.F32 else torch.float64
    g = torch.rand(shape[0] * shape[1], device="cuda", dtype=dt, generator=gen)
    x = torch.rand((g.numel(), m), device="cuda", dtype=dt, generator=gen)
    op = gsf.Operator("gf", shape, g, radius=radius, eps=1e-2, prec=prec)
    y = op.apply(x, gsf.FORM_N)
    first = (2 * (31 + radius) + 1) * shape[1]
    for v in (1e6, float("nan")):
        x[:shape[1]] = v
        assert torch.equal(op.apply(x, gsf.FORM_N)[first:], y[first:]), v


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("rows,radius", [(33, 8), (34, 1), (40, 2), (47, 3), (51, 4), (52, 8), (70, 5)])
def test_gf_block_renewed_sums(gsf, rows, radius, prec):
    """Chunks of more than 32 rows, whose sums are renewed every 2r + 1 rows:
    chunk heights on both sides of a renewal, against the pairs of columns that
    the kernel for other block sizes takes.  Both sum at most a few hundred
    terms in FP64: within 1e-13 (FP64 data), or one unit of the last place of
    the stored coefficients and outputs (FP32)."""
    import torch
    cols = 512 * 254
    gen = torch.Generator(device="cuda").manual_seed(rows)
    dt = torch.float32 if prec == gsf.F32 else torch.float64
    g = torch.rand(rows * cols, device="cuda", dtype=dt, generator=gen)
    x = torch.rand((g.numel(), 4), device="cuda", dtype=dt, generator=gen)
    op = gsf.Operator("gf", (rows, cols), g, radius=radius, eps=1e-2, prec=prec)
    y = op.apply(x, gsf.FORM_N)
    for c in (0, 2):
        ref = op.apply(x[:, c:c + 2].contiguous(), gsf.FORM_N)
        assert (y[:, c:c + 2] - ref).abs().max() <= (1e-13 if prec else 1e-6) * ref.abs().max()


@pytest.mark.parametrize("shape", [(204, 1024), (208, 1024), (512, 512), (624, 624), (632, 624), (640, 720)])
def test_gf_block_small_grids_f64(gsf, shape):
    """Blocks of 4 FP64 columns at r = 8 where the choice between the kernels lies
    at 256 workgroups of the one and 1024 waves of the other, on both sides."""
    test_gf_block_strips(gsf, shape, 8, 4, gsf.F64)


@pytest.mark.parametrize("prec,m", [(0, 4), (0, 8), (1, 4), (1, 8)])
@pytest.mark.parametrize("shape,radius", [((2560, 31), 8), ((2561, 31), 8), ((5200, 60), 8), ((5200, 59), 8),
                                          ((5200, 136), 8), ((5200, 164), 8), ((5200, 193), 8), ((2600, 300), 2),
                                          ((2600, 390), 8), ((20000, 3), 1)])
def test_gf_block_either_kernel(gsf, shape, radius, m, prec):
    """Heights and widths on both sides of the choice of kernel for blocks of 4
    and 8 columns, against the apply of column pairs, whose kernel never
    changes; bounds as above."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(m)
    dt = torch.float32 if prec == gsf.F32 else torch.float64
    g = torch.rand(shape[0] * shape[1], device="cuda", dtype=dt, generator=gen)
    x = torch.rand((g.numel(), m), device="cuda", dtype=dt, generator=gen)
    op = gsf.Operator("gf", shape, g, radius=radius, eps=1e-2, prec=prec)
    y = op.apply(x, gsf.FORM_N)
    for c in range(0, m, 2):
        ref = op.apply(x[:, c:c + 2].contiguous(), gsf.FORM_N)
        assert (y[:, c:c + 2] - ref).abs().max() <= (1e-13 if prec else 1e-6) * ref.abs().max()


@pytest.mark.parametrize("prec,m", [(0, 1), (0, 2), (1, 1)])
@pytest.mark.parametrize("constraint", [False, True])
def test_lobpcg_narrow_block_off_grid(gsf, prec, m, constraint):
    """LOBPCG with rows of less than 16 bytes in a workspace off the 16-byte
    grid, where the update takes a point at a time."""
    import torch
    shape = (25, 41)
    x = _round(scene_2d(*shape, 0.05, 9)[1], prec, gsf)
    p = dict(radius=2, sigma_d=2.0, sigma_r=0.2)
    op = gsf.Operator("bf", shape, _torch(x.ravel(), prec, gsf), prec=prec, **p)
    need = op.workspace(gsf.METHOD_LOBPCG, m).numel()
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")[8:8 + need]
    y, info = op.lobpcg_filter(_torch(x.ravel(), prec, gsf), m, 6, constraint=constraint, ws=ws)
    ref = lobpcg_reference("bf", p, x, shape, m, 6, prec, constraint=constraint)
    check_lobpcg(info, y.cpu().numpy(), ref, m, prec, f"off grid m={m} c={constraint}")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m", [4, 8])
def test_gf_block_operator_off_grid(gsf, m, prec):
    """The GF apply of 4 and 8 columns with the operator's workspace (which holds
    the coefficients between the two passes) off the 16-byte grid."""
    import torch
    shape, radius = (70, 255), 3
    rng = np.random.default_rng(m)
    g = _round(rng.uniform(0.0, 1.0, shape), prec, gsf)
    x = _round(rng.standard_normal((g.size, m)), prec, gsf)
    need = gsf.Operator("gf", shape, _torch(g.ravel(), prec, gsf), radius=radius, eps=1e-2, prec=prec).ws.numel()
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")[8:8 + need]
    op = gsf.Operator("gf", shape, _torch(g.ravel(), prec, gsf), radius=radius, eps=1e-2, prec=prec, ws=ws)
    assert op.ws.data_ptr() == ws.data_ptr()
    ref = oracle.build_operator("gf", g, radius, eps=1e-2)
    for form in (gsf.FORM_N, gsf.FORM_LSYM, gsf.FORM_RW, gsf.FORM_L):
        y = op.apply(_torch(x, prec, gsf), form).cpu().numpy()
        for j in (0, m - 1):
            r = ref.apply(form, x[:, j])
            e = np.linalg.norm(y[:, j] - r) / max(np.linalg.norm(r), np.linalg.norm(x[:, j]))
            assert e <= TOL[prec], (form, j, e)


@pytest.mark.parametrize("prec", [0, 1])
def test_lobpcg_soft_locking_parity(gsf, prec):
    """LOBPCG to a tolerance, where columns reach it at different steps and
    are soft-locked (their W columns count as zero): the GPU stops at the
    oracle's step with the same drop count (where the oracle's reversed run
    agrees) and the same Ritz values, and its output meets the FP64 band gate
    or the FP32 bar."""
    shape, seed = (20, 20), 3
    g = scene_2d(*shape, 0.05, seed)[1]
    par = dict(radius=2, sigma_d=2.0, sigma_r=0.3)
    gr = _round(g, prec, gsf)
    tol = 1e-9 if prec == 1 else 1e-5
    op = gsf.Operator("bf", shape, _torch(gr.ravel(), prec, gsf), **par, prec=prec)
    y, info = op.lobpcg_filter(_torch(gr.ravel(), prec, gsf), 3, 500, tol=tol)

    def run(gg):
        o = oracle.build_operator("bf", gg, 2, 2.0, 0.3)
        yy, th, _, rinfo = oracle.lobpcg_filter(o, gg.ravel(), 3, 500, tol=tol,
                                                data_prec="f64" if prec == 1 else "f32")
        return yy, (th, rinfo)
    ref = reference(run, gr)
    th, rinfo = ref.extra
    e = rel(y.cpu().numpy(), ref.y)
    print(f"soft locking prec={prec}: iters {info.iters}/{rinfo.iters}, dropped {info.dropped}/{rinfo.dropped} "
          f"(reversed {ref.extra_reversed[1].dropped}), y rel {e:.2e}")
    assert info.status == gsf.OK and rinfo.status == "ok"
    assert sum(rinfo.drop_history) > 0
    if prec == 1:
        assert info.iters == rinfo.iters
        if rinfo.dropped == ref.extra_reversed[1].dropped:
            assert info.dropped == rinfo.dropped
        assert e <= ref.gate
        np.testing.assert_allclose(np.array(list(info.theta)[:3]), th, rtol=1e-9, atol=1e-13)
    else:
        assert abs(info.iters - rinfo.iters) <= 3
        assert e <= 1e-5
