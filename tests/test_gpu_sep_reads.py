"""Separable steps on axes of different footprints, in a workspace full of NaN.

The kernels read whole classes of columns; those past an axis' own footprint
carry no weight, so their records must be ones that the slope pass wrote.  Here
the grid goes on beyond the disc or ball on the axis of the short footprint, the
short axis is periodic and about as long as the class, and every byte of the
workspace is 0xFF before the plan's tables go into it.  Bars as in the tests of
the classes' edges: a step 1e-12 (FP64) and 1e-5 (FP32) of the oracle's, a
gradient 1e-10 and 1e-4 of its largest entry."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_14561_amd import Plan, load  # noqa: E402


def _poison(plan):
    """Fill the workspace with 0xFF (NaN in both precisions), then attach it
    again."""
    nbytes = int(plan.info.workspace_bytes)
    plan.workspace.fill_(255)
    base = (plan.workspace.data_ptr() + 255) // 256 * 256
    st = load().fk_plan_set_workspace(plan._h, ctypes.c_void_p(base), max(nbytes, 256),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    return plan


def _S(L, q, h):
    """Scale whose landing points spread over L - 2.5 cells of width h."""
    return (L - 2.5) * h / (2.0 * np.abs(np.polynomial.hermite.hermgauss(q)[0]).max())


def _grid(spec, L, q, region="box", radius=0.0, coef=(), dt=1e-3):
    """Constant drift on axes (n, h, periodic), the spread from the finest."""
    axes = [W.uniform_axis(0.0, (n - 1) * h, n, periodic=per) for n, h, per in spec]
    h = min(s[1] for s in spec)
    p = W.Problem(axes=axes, coef_kind="const", coef=coef or (0.2,) * len(axes), D=float(_S(L, q, h) ** 2 / (4 * dt)),
                  gh_q=q, dt=dt, n_steps=2)
    if region == "ball":
        c = [0.4 * (s[0] - 1) * s[1] for s in spec]
        p = p.replace(region_kind="ball", center=tuple(c + [0.0] * (3 - len(c))), radius=radius)
    return p


CASES = {
    # class 6 from footprints of 4, records to just past the disc
    "disc_4": lambda: W.cell2d(nx=401, ny=201, A=0.5, D=2e-4, dt=1e-3, gh_q=8, n_steps=2),
    "disc_15x4": lambda: _grid([(401, 0.0025, False), (81, 0.0125 * 2, False)], 15, 8, "ball", 0.3),
    "disc_4x12": lambda: _grid([(81, 0.02, False), (301, 0.0025, False)], 12, 8, "ball", 0.25),
    "ball_12x12x3": lambda: _grid([(41, 0.02, False), (41, 0.02, False), (31, 0.3, False)], 12, 5, "ball", 0.3),
    "ball_9x3x4": lambda: _grid([(71, 0.01, False), (21, 0.08, False), (31, 0.06, False)], 9, 6, "ball", 0.25),
    "periodic_15x3": lambda: _grid([(61, 0.01, False), (9, 0.16, True)], 15, 8),
    "periodic_12x12x3": lambda: _grid([(31, 0.01, False), (27, 0.01, False), (8, 0.16, True)], 12, 5),
}


@pytest.mark.parametrize("prec,bar", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_step(name, prec, bar):
    p = CASES[name]()
    u = W.random_field(p.shape, 7)
    for a, ax in enumerate(p.axes):   # images hold their originals' values
        if ax.periodic:
            v = np.moveaxis(u, a, 0)
            v[-1] = v[0]
    plan = _poison(Plan(p, precision=prec, step_kernel="box"))
    got = plan.split(plan.step(1, torch.from_numpy(u.reshape(-1))))[0].double().cpu().numpy()
    own = plan.split(plan.forward([0]))[0].double().cpu().numpy()[0]
    assert plan.check_flags() == 0
    plan.close()
    assert np.abs(got - oracle.step(p, 1, u)).max() <= bar
    assert np.abs(own - oracle.solve(p, snaps=[0])[0]).max() <= bar


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_gradient(name, prec, bar):
    p = CASES[name]()
    lam = W.region_mean_weights(p)
    g_ref, _ = oracle.adjoint(p, lam)
    plan = _poison(Plan(p, precision=prec, ckpt_every=1))
    g, _ = plan.adjoint(torch.from_numpy(lam.reshape(-1)))
    g = g.cpu().numpy()[0]
    plan.close()
    assert np.abs(g - g_ref).max() <= bar * np.abs(g_ref).max(), (g, g_ref)
