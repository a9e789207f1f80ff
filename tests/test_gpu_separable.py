"""The separable and one-launch steps, and their transposes, at the edges of
their footprint classes, on odd grids, against the oracle.

2D footprints 5 .. 15 nodes per axis (classes 6, 9, 12, 15) and past them, 3D
3 .. 12 and past; faces, a disc, periodic axes; every compiled Q* of the
one-launch step.  One step from a random field: FP64 within 1e-12, FP32 within
1e-5 of the oracle (the stated bars).  Gradients over a few steps: 1e-10 of the
largest entry in FP64, 1e-4 in FP32."""
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


def _spread(L, q, h, dt):
    """Diffusion whose landing points spread over L - 2.5 cells of width h."""
    a = np.abs(np.polynomial.hermite.hermgauss(q)[0]).max()
    S = (L - 2.5) * h / (2.0 * a)
    return float((S / 2.0) ** 2 / dt)


def _flow2d(L, region, q=8, n=(71, 45), steps=3):
    h, dt = 1.0 / (n[1] - 1), 1e-3
    axes = [W.uniform_axis(0.0, (n[0] - 1) * h, n[0]), W.uniform_axis(0.0, 1.0, n[1])]
    p = W.Problem(axes=axes, coef_kind="cellular2d", coef=(4.0, 0.2, 5.0), D=_spread(L, q, h, dt), gh_q=q, dt=dt,
                  n_steps=steps)
    if region == "ball":
        p = p.replace(region_kind="ball", center=(0.75, 0.5, 0.0), radius=0.47)
    return p


def _rolls(L, q=6, n=(67, 37), steps=3):
    h = 1.0 / (n[1] - 1)
    dt = 5e-4
    return W.Problem(axes=[W.uniform_axis(0.0, 66 * h, n[0], periodic=True), W.uniform_axis(0.0, 1.0, n[1])],
                     coef_kind="rolls2d", coef=(8.0, 0.2, 0.7, 2.0), D=_spread(L, q, h, dt), gh_q=q, dt=dt, n_steps=steps)


def _abc(L, q=4, n=27, steps=2):
    p = W.abc3d(n=n, gh_q=q, dt=0.02, n_steps=steps)
    h = float(np.diff(p.axes[2].nodes).min())
    return p.replace(D=_spread(L, q, h, 0.02))


def _field(p, seed=5):
    u = W.random_field(p.shape, seed)
    for a, ax in enumerate(p.axes):   # images hold their originals' values
        if ax.periodic:
            ix = [slice(None)] * p.d
            first = list(ix)
            ix[a], first[a] = -1, 0
            u[tuple(ix)] = u[tuple(first)]
    return u


def _check_step(p, prec, kernel, hermite="r1"):
    u = _field(p)
    ref = oracle.step(p.replace(hermite=hermite), 1, u)
    plan = Plan(p, precision=prec, step_kernel=kernel, hermite=hermite)
    got = plan.split(plan.step(1, torch.from_numpy(u.reshape(-1))))[0].double().cpu().numpy()
    own = plan.split(plan.forward([0]))[0].double().cpu().numpy()[0]
    assert plan.check_flags() == 0
    plan.close()
    err = np.abs(got - ref).max()
    assert err <= BAR[prec], err
    # periodic plans take a caller's field per point and their own as the class says
    err = np.abs(own - oracle.solve(p.replace(hermite=hermite), snaps=[0])[0]).max()
    assert err <= BAR[prec], err


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("region", ["box", "ball"])
@pytest.mark.parametrize("L", [3, 5, 6, 7, 9, 10, 12, 13, 15, 16, 19])
def test_step_2d(L, region, prec):
    _check_step(_flow2d(L, region), prec, "box")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L,hermite", [(4, "r1"), (9, "r1"), (14, "r2"), (6, "r2")])
def test_step_2d_periodic(L, hermite, prec):
    _check_step(_rolls(L), prec, "box", hermite)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L", [3, 4, 5, 6, 8, 9, 11, 12, 13])
def test_step_3d(L, prec):
    _check_step(_abc(L), prec, "box")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("q", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("region,L", [("box", 5), ("ball", 9), ("ball", 24), ("periodic", 6)])
def test_one_launch_step_2d(region, L, q, prec):
    """L = 24: a patch and its reach hold more records than the one-launch step
    takes, the two-launch step runs."""
    p = _rolls(L, q) if region == "periodic" else _flow2d(L, region, q)
    _check_step(p, prec, "auto")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("hermite", ["r1", "r2"])
@pytest.mark.parametrize("name", ["rolls", "abc", "abc_wide"])
def test_caller_fields_with_other_values_on_image_nodes(name, hermite, prec):
    """A caller's field is read node by node: its image nodes need not hold
    their originals' values."""
    p = {"rolls": _rolls(6), "abc": _abc(4, n=19), "abc_wide": _abc(7, n=23)}[name]
    u = W.random_field(p.shape, 9)
    ref = oracle.step(p.replace(hermite=hermite), 1, u)
    plan = Plan(p, precision=prec, hermite=hermite)
    got = plan.split(plan.step(1, torch.from_numpy(u.reshape(-1))))[0].double().cpu().numpy()
    frm = plan.split(plan.forward_from(torch.from_numpy(u.reshape(-1)), 2, [1]))[0].double().cpu().numpy()[0]
    plan.close()
    assert np.abs(got - ref).max() <= BAR[prec] and np.abs(frm - ref).max() <= BAR[prec]


@pytest.mark.parametrize("q", [4, 7])
def test_one_launch_step_2d_r2(q):
    _check_step(_flow2d(7, "ball", q), "f64", "auto", "r2")


def _check_gradient(p, prec, bar, kernel="auto"):
    lam = W.region_mean_weights(p)
    g_ref, _ = oracle.adjoint(p, lam)
    plan = Plan(p, precision=prec, ckpt_every=2, step_kernel=kernel)
    if kernel == "box":
        assert plan.info.adj_box_nodes > 0
    g, _ = plan.adjoint(torch.from_numpy(lam.reshape(-1)))
    g = g.cpu().numpy()[0]
    plan.close()
    err = np.abs(g - g_ref).max() / np.abs(g_ref).max()
    assert err <= bar, (err, g, g_ref)


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("L", [3, 5, 6, 9, 10, 12, 13, 15, 16, 19])
def test_gradient_2d(L, prec, bar):
    _check_gradient(_flow2d(L, "ball"), prec, bar)


@pytest.mark.parametrize("L", [4, 8])
def test_gradient_2d_periodic(L):
    _check_gradient(_rolls(L), "f64", 1e-10)


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("L", [3, 4, 6, 7, 9, 12, 13])
def test_gradient_3d(L, prec, bar):
    _check_gradient(_abc(L), prec, bar)


@pytest.mark.parametrize("prec,bar", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("name,L", [("flow", 5), ("flow", 14), ("flow", 18), ("abc", 3), ("abc", 7)])
def test_transposed_step_is_the_transpose(name, L, prec, bar):
    """<A x, y> = <x, A^T y> with the two sides' own kernels, over the sum of
    the terms' sizes."""
    p = _flow2d(L, "ball") if name == "flow" else _abc(L)
    plan = Plan(p, precision=prec, ckpt_every=1, step_kernel="box")
    rng = np.random.default_rng(8)
    x = np.stack([_field(p, 20 + f).reshape(-1) for f in range(p.d + 1)])
    y = rng.uniform(-1.0, 1.0, size=p.n_nodes)
    ax = plan.apply_step(1, torch.from_numpy(x)).double().cpu().numpy()
    aty = plan.apply_step(1, torch.from_numpy(y), transpose=True).double().cpu().numpy()
    plan.close()
    lhs, rhs = float((ax * y).sum()), float((x * aty).sum())
    assert abs(lhs - rhs) <= bar * float((np.abs(x) * np.abs(aty)).sum())


@pytest.mark.parametrize("prec,bar", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("kernel", ["auto", "split", "box"])
@pytest.mark.parametrize("name,L", [("rolls", 4), ("rolls", 9), ("rolls", 14), ("abc", 3), ("abc", 9)])
def test_transposed_step_with_image_nodes_of_their_own(name, L, kernel, prec, bar):
    """The same on periodic axes with fields whose images hold other values than
    their originals: both sides take them as the same nodes."""
    p = _rolls(L) if name == "rolls" else _abc(L, n=23)
    plan = Plan(p, precision=prec, ckpt_every=1, step_kernel=kernel)
    rng = np.random.default_rng(11)
    x = rng.uniform(-1.0, 1.0, size=(p.d + 1, p.n_nodes))
    y = rng.uniform(-1.0, 1.0, size=p.n_nodes)
    ax = plan.apply_step(1, torch.from_numpy(x)).double().cpu().numpy()
    aty = plan.apply_step(1, torch.from_numpy(y), transpose=True).double().cpu().numpy()
    plan.close()
    lhs, rhs = float((ax * y).sum()), float((x * aty).sum())
    assert abs(lhs - rhs) <= bar * float((np.abs(x) * np.abs(aty)).sum())


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("flow,L", [("2d", 9), ("2d", 12), ("2d", 13), ("2d", 15), ("3d", 6), ("3d", 9), ("3d", 12)])
def test_gradient_in_separable_form(flow, L, prec, bar):
    """The classes' transposed steps also where a default plan goes per landing
    point (footprints wide beside Q*)."""
    _check_gradient(_flow2d(L, "ball") if flow == "2d" else _abc(L), prec, bar, "box")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("q,L,region", [(2, 6, "box"), (3, 5, "ball"), (3, 9, "box"), (6, 8, "ball"), (6, 11, "box")])
def test_default_layouts_3d(q, L, region, prec):
    """Default plans on both sides of the rule between separable nodes and points
    by lanes or threads."""
    h = 1.0 / 22
    p = W.Problem(axes=[W.uniform_axis(0.0, 22 * h, n) for n in (23, 21, 25)], coef_kind="const",
                  coef=(0.3, -0.2, 0.1), D=_spread(L, q, h, 1e-3), gh_q=q, dt=1e-3, n_steps=2)
    if region == "ball":
        p = p.replace(region_kind="ball", center=(0.5, 0.5, 0.5), radius=0.46)
    _check_step(p, prec, "auto")
