"""The assembled product with four lanes per row (plans of up to a quarter of a
million rows) against the oracle: row counts at the edges of its 64-row parts,
one to eight columns in storage order and out of it, boxes whose value blocks do
not divide by four, a grid on the other side of the rule."""
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


def _problem(d, n, D, q=4):
    ax = [W.uniform_axis(0.0, 1.0, k) for k in n]
    return W.Problem(axes=ax, coef_kind="const", coef=(0.7, -0.4, 0.2)[:d], D=D, region_kind="box", gh_q=q, dt=0.01,
                     n_steps=5)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("d,n", [(1, (6,)), (1, (66,)), (1, (67,)), (1, (259,)), (2, (10, 10)), (2, (18, 6)),
                                 (2, (19, 34)), (3, (5, 6, 7)), (3, (8, 9, 12))])
@pytest.mark.parametrize("D", [1e-5, 3e-2])
def test_pass_at_the_edges_of_the_parts(d, n, D, prec):
    p = _problem(d, n, D)
    plan = Plan(p, precision=prec, form="ell")
    got = plan.split(plan.forward([0]))[0].double().cpu().numpy()[0]
    assert plan.check_flags() == 0
    plan.close()
    assert np.abs(got - oracle.solve(p, snaps=[0])[0]).max() <= BAR[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("columns", [1, 2, 3, 4])
@pytest.mark.parametrize("horizons", [[5], [1, 2, 3, 4, 5], [5, 1, 4, 2, 3, 5, 5, 5]])
def test_columns(horizons, columns, prec):
    p = _problem(2, (21, 17), 4e-3)
    plan = Plan(p, precision=prec, form="ell", columns=columns)
    got = plan.split(plan.forward_horizons(horizons))[0].double().cpu().numpy()
    assert plan.check_flags() == 0
    plan.close()
    assert np.abs(got - oracle.solve_horizons(p, horizons)).max() <= BAR[prec]


def test_a_lane_per_row_on_the_other_side():
    """0.28 million rows: 1024 and more work items of 256 rows."""
    p = _problem(2, (533, 533), 1e-6, q=3).replace(n_steps=2)
    plan = Plan(p, form="ell", columns=2)
    got = plan.split(plan.forward_horizons([1, 2]))[0].cpu().numpy()
    plan.close()
    assert np.abs(got - oracle.solve_horizons(p, [1, 2])).max() <= BAR["f64"]
