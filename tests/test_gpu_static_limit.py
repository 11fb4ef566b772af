"""Problems at the limit of the static workspace run there with what fits: 1D steps with a launch per
stage instead of whole (bit for bit the same states, time steps and switch decisions, the limiter
acting), triangles and 2D meshes as they are; and the workspace that a context reports is the one it
uses."""

import numpy as np
import pytest

from gpu_util import RTOL_FP64, announce, oracle_for, rel_l2, to_dev, to_np
from oracle import stabilize as ost
from oracle.initial import project_initial
from paper_2112_05946_amd import inputs
from paper_2112_05946_amd.binding import Solver

pytestmark = pytest.mark.gpu

STATIC = 64 << 20


def _run(cfg, u0, static, n, dt=None):
    """n steps in one call, or one by one at a fixed dt."""
    import torch
    sol = Solver(cfg, static_workspace=static)
    sol.timing(True)
    u = to_dev(u0)
    dts = torch.empty(n, dtype=torch.float64, device="cuda")
    flags = torch.empty(4 * sol.E * n, dtype=torch.uint8, device="cuda")
    if dt is None:
        sol.steps(u, n, dts, flags)
    else:
        for i in range(n):
            sol.step(u, dt, dts[i:i + 1], flags[4 * sol.E * i:4 * sol.E * (i + 1)])
    sol.sync()
    passes, used = set(sol.timing_read()), sol.info["workspace_bytes"]
    sol.close()
    return to_np(u), to_np(dts), to_np(flags), passes, used


@pytest.mark.parametrize("start", ["initial", "near_vacuum"])
@pytest.mark.parametrize("label,cfg", [("sod", inputs.small(inputs.SOD, 8523)), ("sod_hll", inputs.small(inputs.SOD_HLL, 8523)),
                                       ("sod_hll_bs3", inputs.small(inputs.SOD_HLL_BS3, 6077)),
                                       ("burgers", inputs.small(inputs.BURGERS, 22540))])
def test_whole_steps_equal_a_launch_per_stage(label, cfg, start):
    announce("static_limit", label, start)
    prob, (T, R) = oracle_for(cfg)
    dt = None
    if start == "initial":
        u0 = project_initial(prob, cfg["ic"], (T, R))
    elif prob.S > 1:  # (at a CFL step such a state can lose its means)
        u0 = ost.limit(prob, T, R, inputs.fuzz_euler(1, R.M, prob.E, prob.nsp, 3, vacuum_frac=0.3))[0]
        dt = 1e-6
    else:
        u0 = inputs.fuzz_scalar(R.M, prob.E, prob.nsp, 3, scale=0.1, offset=0.8)
    u, du, fu, pu, _ = _run(cfg, u0, False, 3, dt)
    v, dv, fv, pv, used = _run(cfg, u0, True, 3, dt)
    assert pu <= {"cfl", "copy", "stage1"} and len(pv - {"cfl"}) > 1, (pu, pv)
    assert used <= STATIC
    assert np.array_equal(du, dv) and np.array_equal(fu, fv) and np.array_equal(u, v)
    if prob.S > 1 and start == "near_vacuum":
        assert fu.reshape(3, 4, -1)[:, 0].any()


def test_2d_workspace_in_use():
    """60 x 25 elements, bs3: without room for its face traces (those of the 4 x 2 tiles would fit)."""
    cfg = dict(inputs.small(inputs.SHOCK_VORTEX, 60, 25), integrator="bs3")
    prob, (T, R) = oracle_for(cfg)
    u0 = project_initial(prob, cfg["ic"], (T, R))
    u, _, _, _, need = _run(cfg, u0, False, 2)
    v, _, _, _, used = _run(cfg, u0, True, 2)
    assert used <= STATIC < need
    assert rel_l2(v, u) < RTOL_FP64


def test_triangles_at_the_limit():
    n = 7802
    rng = np.random.default_rng(5)
    xy = np.array([[0.0, 0.0], [1.0, 0.0], [0.0, 1.0]]) + 0.1 * rng.random((n, 3, 2))
    mesh = dict(xy=xy, nbr=np.full((n, 3), -1, np.int32), nbr_face=np.full((n, 3), -1, np.int32))
    cfg = dict(inputs.tri_shock_vortex(4), p=3, gpc_order=2, nq1d=3, mesh=mesh, bc=["outflow"] * 4)
    u0 = inputs.fuzz_euler(2, 6, n, 10, 3)
    u, du, fu, _, need = _run(cfg, u0, False, 2)
    v, dv, fv, _, used = _run(cfg, u0, True, 2)
    assert used == need and STATIC < used <= STATIC + (8 << 10)
    assert np.array_equal(u, v) and np.array_equal(du, dv) and np.array_equal(fu, fv)
