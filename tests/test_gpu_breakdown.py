"""Breakdown of the CG filters through p^T q at a step later than the first,
with many workgroups: every workgroup of the update sums p^T q itself, so all
of them have to stop in the same step and the last iterate has to come back.

The signals make p^T q of step 2 zero in exact IEEE arithmetic.  The image
consists of horizontal pairs of pixels whose guidance lies 50 sigma_r and more
from every neighbouring pair's (weights of exp(-1250) = 0), so the graph is a
set of 2 x 2 blocks with one non-zero eigenvalue each: l1 = 0.76 for the pairs
of the upper half (equal guidance), l2 below 1e-3 for those of the lower half.
The residual's components are 1e-150 and 1e-161: step 1 removes the first up
to rounding (1e-166), r^T r of step 2 then holds the squares 1e-322 of the
second, above the breakdown floor, and the products l2 1e-322 of p^T q are
below half the smallest positive number."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
SHAPE = (256, 384)   # 384 vector workgroups of 256 points


def _pairs(delta):
    """Guidance in units of sigma_r (pairs of equal values above, delta apart
    below) and the pairs' +1 / -1 pattern with random signs."""
    rows, cols = SHAPE
    y, x = np.indices(SHAPE)
    level = 50.0 * (2 * (y % 2) + (x // 2) % 2)
    side = 1.0 - 2.0 * (x % 2)
    lower = y >= rows // 2
    sign = np.repeat(np.random.default_rng(4).choice([-1.0, 1.0], (rows, cols // 2)), 2, axis=1)
    return level + lower * (0.5 * delta) * side, side * sign, lower


def _dev(x):
    import torch
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _linear():
    g, e, lower = _pairs(3.8)     # w = exp(-0.5 - 3.8^2 / 2) = 4.4e-4 in the lower pairs
    w = np.exp(-0.5 - 0.5 * 3.8 ** 2)
    x0 = e * np.where(lower, 1e-161 * (1.0 + w) / (2.0 * w), 1e-150)
    par = dict(radius=1, sigma_d=1.0, sigma_r=1.0)
    ref = oracle.build_operator("bf", g, 1, 1.0, 1.0)
    y, info = oracle.cg_filter_normalized(ref, x0.ravel(), 6)
    assert info.status == "breakdown" and info.iters == 1
    return g, x0.ravel(), par, y, lower.ravel()


def _check(x, one, ref, lower):
    import torch
    assert torch.equal(x, one)    # the iterate of step 1, to the bit
    x = x.cpu().numpy()
    assert np.abs(x[~lower]).max() <= 1e-12 * 1e-150
    assert np.abs(x[lower] - ref[lower]).max() <= 1e-12 * np.abs(ref[lower]).max()


@pytest.mark.parametrize("m", [0, 1, 3])
def test_cg_stops_at_step_two(gsf, m):
    """m = 0: the single-column filter; else the block filter, all columns."""
    g, x0, par, ref, lower = _linear()
    op = gsf.Operator("bf", SHAPE, _dev(g.ravel()), prec=gsf.F64, **par)
    if m == 0:
        x, info = op.cg_filter(_dev(x0), 6)
        one, info1 = op.cg_filter(_dev(x0), 1)
        assert (info.status, info.iters) == (gsf.EBREAKDOWN, 1) and info1.status == gsf.OK
        _check(x, one, ref, lower)
        return
    X0 = _dev(np.stack([x0] * m, axis=1))
    X, infos = op.cg_filter_block(X0, 6)
    one, _ = op.cg_filter_block(X0, 1)
    for c in range(m):
        assert (infos[c].status, infos[c].iters) == (gsf.EBREAKDOWN, 1)
        _check(X[:, c].contiguous(), one[:, c].contiguous(), ref, lower)


def test_block_columns_stop_alone(gsf):
    """A column that stops leaves the others running."""
    g, x0, par, ref, lower = _linear()
    op = gsf.Operator("bf", SHAPE, _dev(g.ravel()), prec=gsf.F64, **par)
    other = np.random.default_rng(8).standard_normal(x0.size)
    X, infos = op.cg_filter_block(_dev(np.stack([other, x0], axis=1)), 2)
    one, _ = op.cg_filter_block(_dev(np.stack([other, x0], axis=1)), 1)
    assert (infos[1].status, infos[1].iters) == (gsf.EBREAKDOWN, 1)
    _check(X[:, 1].contiguous(), one[:, 1].contiguous(), ref, lower)
    y, info = op.cg_filter(_dev(other), 2)
    assert infos[0].iters == info.iters == 2
    assert (X[:, 0] - y).abs().max() <= 1e-12 * y.abs().max()


def test_joint_cg_stops_at_step_two(gsf):
    """The update phase as extra workgroups of the Rayleigh-Ritz launch."""
    g, x0, par, ref, lower = _linear()
    op = gsf.Operator("bf", SHAPE, _dev(g.ravel()), prec=gsf.F64, **par)
    lob = _dev(np.random.default_rng(9).standard_normal(x0.size))
    x, y, ci, li = op.joint_filter(_dev(x0), 6, lob, 4, 6)
    one = op.cg_filter(_dev(x0), 1)[0]
    assert (ci.status, ci.iters) == (gsf.EBREAKDOWN, 1) and li.iters == 6
    x = x.cpu().numpy()
    assert np.abs(x[~lower]).max() <= 1e-12 * 1e-150
    assert np.abs(x - one.cpu().numpy()).max() <= 1e-12 * np.abs(x).max()
    assert np.isfinite(y.cpu().numpy()).all()


def test_reguided_cg_stops_at_step_two(gsf):
    """The same pattern with the iterate as the guidance: pairs one sigma_r
    apart above (removed by step 1) and 7 apart below (w = 1.4e-11: residual
    1e-10, squares 1e-320, products 1e-331)."""
    import torch
    sr = 1e-150
    g, e, lower = _pairs(7.0)
    side = 1.0 - 2.0 * (np.indices(SHAPE)[1] % 2)
    x0 = (sr * (g + 0.5 * side * ~lower)).ravel()
    ref, rinfo = oracle.cg_filter_reguided("bf", x0, SHAPE, 6, 1, 1.0, sr)
    assert rinfo.status == "breakdown" and rinfo.iters == 1
    kw = dict(radius=1, sigma_d=1.0, sigma_r=sr, prec=gsf.F64)
    x, info = gsf.reguided_filter("bf", SHAPE, _dev(x0), gsf.METHOD_CG, 6, **kw)
    one, _ = gsf.reguided_filter("bf", SHAPE, _dev(x0), gsf.METHOD_CG, 1, **kw)
    assert (info.status, info.iters) == (gsf.EBREAKDOWN, 1)
    assert torch.equal(x, one)
    assert np.abs(x.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
