"""fk_tune times every layout a plan can run: the one of the default among them,
the thread per node apart from the lane groups and the entry form."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_14561_amd import Plan, tune  # noqa: E402

CASES = {
    "line": (lambda: W.bm1d(n_steps=64), {"node", "split", "group"}),
    "one_launch": (lambda: W.paper2d(), {"node", "split", "group"}),
    "abc": (lambda: W.abc3d(n=25, n_steps=8), {"node", "split", "group", "box"}),
    "runaway": (lambda: W.runaway3d(n_p=33, n_xi=33, T=2.0), {"node", "split", "group", "box"}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_tuned_layouts(name):
    prob, layouts = CASES[name][0](), CASES[name][1]
    res = tune(prob, precision="f32", trial_steps=64)
    assert layouts <= set(res["ms_per_step"]), res
    assert res["ms_per_step"][res["step_kernel"]] == min(res["ms_per_step"].values())
    if name == "line":   # many steps to a launch against two launches a step
        assert res["step_kernel"] == "split" and res["ms_per_step"]["split"] < 0.5 * res["ms_per_step"]["node"]
    # the layouts are ones of the same scheme
    ref = None
    for k in res["ms_per_step"]:
        plan = Plan(prob, precision="f32", step_kernel=k)
        u = plan.forward([0])[0].double().cpu().numpy()
        plan.close()
        ref = u if ref is None else ref
        assert np.abs(u - ref).max() <= 2e-5, k
