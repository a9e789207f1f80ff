"""fk_forward_from: the caller's state is read by its own step only.  Exit nodes of
that state may hold any value; those of every later field hold the scheme's.
Snapshots of several steps against the oracle's, step by step (FP64 1e-12, FP32
1e-5; an instance computed in FP64 inside an FP32 plan as FP32)."""
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

CASES = {
    "line": lambda: W.bm1d(n=101, n_steps=6, gh_q=8),
    "line_long": lambda: W.bm1d(n=5001, n_steps=6, gh_q=4, dt=1e-4),
    "disc": lambda: W.cell2d(nx=65, ny=33, n_steps=6, D=2e-3),
    "rolls": lambda: W.paper2d(n1=41, n2=17).replace(n_steps=6),
    "abc": lambda: W.abc3d(n=13, n_steps=6, gh_q=3),
    "faces": lambda: W.Problem(axes=[W.uniform_axis(0.0, 1.0, 25), W.uniform_axis(0.0, 1.0, 21)], coef_kind="const",
                               coef=(0.4, -0.3), D=0.05, gh_q=4, dt=5e-3, n_steps=6,
                               faces=(("exit0", "reflect"), ("exit1", "exit0"))),
}


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("prec,bar", [("f64", 1e-12), ("f32", 1e-5), ("mixed", 1e-5)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_exit_nodes_of_the_state(name, prec, bar, use_graph):
    p = CASES[name]()
    force = [1] if prec == "mixed" else None
    u = W.random_field(p.shape, 12)
    refs, r = {5: u}, u
    for m in range(4, -1, -1):
        r = oracle.step(p, m, r)
        refs[m] = r
    plan = Plan(p, precision="f64" if prec == "f64" else "f32", use_graph=use_graph, force_f64=force)
    x = torch.from_numpy(u.reshape(-1)).to("cuda", plan.dtype)
    snaps = [5, 4, 3, 2, 0]
    for _ in range(2):
        got = plan.split(plan.forward_from(x, 5, snaps))[0].double().cpu().numpy()
        for k, m in enumerate(snaps):
            assert np.abs(got[k] - refs[m]).max() <= bar, m
    assert plan.check_flags() == 0
    plan.close()
