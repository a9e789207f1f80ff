"""Values that are not finite in a caller's field reach the nodes whose inside
landing points touch them, and no others: in every step layout the node set that
the oracle (a loop over the points) makes NaN or infinite, and its values
elsewhere (FP64 within 1e-12, FP32 within 1e-5).  (A node whose own value is not
finite may be so too: sums are taken relative to it.)

Fields: NaN or infinity everywhere outside the region (a mask), and at single
nodes inside it."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_14561_amd import Plan  # noqa: E402

BAR = {"f64": 1e-12, "f32": 1e-5}


def _D(L, q, h, dt):
    a = np.abs(np.polynomial.hermite.hermgauss(q)[0]).max()
    return float(((L - 2.5) * h / (2.0 * a)) ** 2 / (4.0 * dt))


def _const(n, L, q, drift, ball=0.0, dt=1e-3, periodic=()):
    h = 1.0 / (n[-1] - 1)
    axes = [W.uniform_axis(0.0, (k - 1) * h, k, periodic=a in periodic) for a, k in enumerate(n)]
    p = W.Problem(axes=axes, coef_kind="const", coef=tuple(c * h / dt for c in drift), D=_D(L, q, h, dt), gh_q=q,
                  dt=dt, n_steps=2)
    if ball:
        c = [0.5 * (k - 1) * h for k in n]
        p = p.replace(region_kind="ball", center=tuple(c + [0.0] * (3 - len(c))), radius=ball)
    return p


# drifts of up to two cells: points of a node far from its own cell
CASES = {
    "line": (_const((101,), 7, 8, (1.3,)), "auto"),
    "line_ball": (_const((201,), 9, 7, (-2.2,), ball=0.4), "auto"),
    "line_long": (_const((301,), 9, 7, (-2.2,), ball=0.4), "auto"),
    "one_launch_box": (_const((61, 47), 5, 6, (1.7, -0.6)), "auto"),
    "one_launch_disc": (_const((61, 47), 9, 4, (1.7, -2.6), ball=0.45), "auto"),
    "separable_2d": (_const((61, 47), 9, 4, (1.7, -2.6)), "box"),
    "separable_2d_gaps": (_const((91, 67), 14, 3, (0.7, 0.4), ball=0.47), "box"),
    "points_2d": (_const((91, 67), 22, 8, (1.7, -2.6), ball=0.47), "box"),
    "separable_3d": (_const((27, 23, 25), 4, 4, (1.3, -0.7, 0.2)), "box"),
    "separable_3d_gaps": (_const((27, 23, 25), 9, 3, (1.3, -0.7, 0.2), ball=0.45), "box"),
    "periodic_3d": (_const((27, 23, 25), 4, 4, (1.3, -0.7, 0.2), periodic=(0, 1)), "auto"),
}


def _compare(got, ref, u, bar):
    fin = np.isfinite(ref) & np.isfinite(u)
    assert not np.isfinite(got[~np.isfinite(ref)]).any()
    assert np.isfinite(got[fin]).all(), int((~np.isfinite(got[fin])).sum())
    assert fin.any() and np.abs(got[fin] - ref[fin]).max() <= bar


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("hermite", ["r1", "r2"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_step_from_a_field_with_values_that_are_not_finite(name, hermite, prec):
    p, kernel = CASES[name]
    if hermite == "r2" and (p.d == 1 or (p.d == 3 and kernel == "box")):
        pytest.skip("not a layout of R2")
    q = p.replace(hermite=hermite)
    plan = Plan(p, precision=prec, step_kernel=kernel, hermite=hermite)
    exits = oracle.solve(p.replace(n_steps=1, D=1e-30, coef=(0.0,) * p.d), snaps=[1])[0] == 1.0
    rng = np.random.default_rng(4)
    for bad in (np.nan, np.inf):
        for where in ("outside", "inside"):
            u = W.random_field(p.shape, 3)
            for a, ax in enumerate(p.axes):
                if ax.periodic:
                    np.moveaxis(u, a, 0)[-1] = np.moveaxis(u, a, 0)[0]
            if where == "outside":
                u[exits] = bad
            else:
                u.reshape(-1)[rng.choice(np.flatnonzero(~exits), 3, replace=False)] = bad
            with np.errstate(all="ignore"):
                ref = oracle.step(q, 1, u)
            got = plan.split(plan.step(1, torch.from_numpy(u.reshape(-1))))[0].double().cpu().numpy()
            _compare(got, ref, u, BAR[prec])
            frm = plan.split(plan.forward_from(torch.from_numpy(u.reshape(-1)), 2, [1]))[0]
            _compare(frm.double().cpu().numpy()[0], ref, u, BAR[prec])
    plan.close()
