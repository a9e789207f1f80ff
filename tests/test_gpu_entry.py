"""The entry form of the 3D step (faces, node-dependent diffusion, axes that
are not uniform) against the oracle and the lane-group step: every compiled
Q*, exit-0, exit-1, reflecting and periodic axes mixed, grids of odd sizes on
both sides of the rule that chooses it, the runaway model with and without the
thermal quench, two fields in one batch, graph replays.  FP64 within 1e-12,
FP32 within 1e-5 of the oracle (the stated bars)."""
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
FACES = (("exit0", "exit1"), ("reflect", "exit0"), ("exit1", "reflect"))


def _run(probs, prec, **kw):
    plan = Plan(probs, precision=prec, use_graph=True, **kw)
    for _ in range(3):
        out = [o.double().cpu().numpy()[0] for o in plan.split(plan.forward([0]))]
        torch.cuda.synchronize()
    assert plan.check_flags() == 0
    plan.close()
    return out


def _check(probs, prec, **kw):
    got = _run(probs, prec, **kw)
    for g, p in zip(got, probs if isinstance(probs, list) else [probs]):
        err = float(np.abs(g - oracle.solve(p, snaps=[0])[0]).max())
        assert err <= BAR[prec], err


def _box(n, q, D, faces, periodic=False, graded=False, steps=3):
    ax = [W.uniform_axis(0.0, 1.0, n[0], periodic=periodic), W.uniform_axis(0.0, 1.0, n[1]),
          W.remark2_axis(0.0, 0.7, 1.0, 1.0 / 20, 1.0 / 60) if graded else W.uniform_axis(0.0, 1.0, n[2])]
    if periodic:
        faces = (("exit1", "exit1"),) + faces[1:]
    return W.Problem(axes=ax, coef_kind="const", coef=(-0.8, 0.5, 0.3), D=D, region_kind="box", gh_q=q, dt=0.01,
                     n_steps=steps, faces=faces)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("q", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("D", [1e-5, 3e-3, 0.05])
def test_mixed_faces_every_order(q, D, prec):
    _check(_box((23, 19, 37), q, D, FACES), prec)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [(5, 4, 7), (29, 31, 33), (47, 53, 65)])
@pytest.mark.parametrize("form", ["faces", "periodic", "graded", "graded_faces"])
def test_sizes_and_axes(n, form, prec):
    exit1 = (("exit1", "exit1"),) * 3
    p = _box(n, 4, 4e-3, exit1 if form == "graded" else FACES, periodic=form == "periodic",
             graded=form.startswith("graded"), steps=2)
    _check(p, prec)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_against_the_lane_group_step(prec):
    p = _box((41, 39, 35), 4, 2e-3, FACES, graded=True, steps=4)
    a, b = _run(p, prec)[0], _run(p, prec, step_kernel="group")[0]
    assert float(np.abs(a - b).max()) <= 2 * BAR[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_runaway_fields_and_quench(prec):
    kw = dict(n_p=17, n_xi=13, dt=0.5, T=4.0)
    a = W.runaway3d(**kw)
    _check([a, W.runaway3d(E=a.coef[0] * 1.5, **kw)], prec)
    _check(W.runaway3d(t_star=2.0, E0=0.05, That0=3.0, Thatf=0.5, Ttilde=3.0, tau=6000.0, **kw), prec)
