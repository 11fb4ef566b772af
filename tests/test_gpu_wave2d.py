"""The FP64 stage kernel with one element per wave where its split can go wrong: meshes of one
element, one short of and one past its 2 x 2 tile, several tiles; 3 x 3 and 4 x 4 points; node
counts that are and are not multiples of the group of four; all boundary kinds; SSP-RK3 stages,
Butcher rows, the filter and the limiter acting, chained steps; and the static workspace with
and without room for the face traces.  Against the oracle at the FP64 parity bar."""

import ctypes

import numpy as np
import pytest

from gpu_util import (ELEM_RTOL, RTOL_FP64, announce, check_flags, elem_max_rel, oracle_for, rel_l2, solver_for, to_dev,
                      to_np)
from oracle import fr as ofr
from oracle import stabilize as ost
from oracle import stepper as ostep
from oracle.initial import project_initial
from paper_2112_05946_amd import binding, inputs

pytestmark = pytest.mark.gpu

# (gpc_order, nq1d, rdim) of (15, 25), (10, 16) and (3, 4) modes and nodes
SIZES = {"m15q25": (4, 5, 2), "m10q16": (3, 4, 2), "m3q4": (2, 4, 1)}
MESHES = [(1, 1), (2, 1), (3, 3), (1, 4), (5, 4)]


def _cfg(nx, ny, p, size, **kw):
    order, nq, rdim = SIZES[size]
    return dict(inputs.small(inputs.SHOCK_VORTEX, nx, ny), p=p, gpc_order=order, nq1d=nq, rdim=rdim, **kw)


@pytest.mark.parametrize("flux", ["rusanov", "hll"])
@pytest.mark.parametrize("size", list(SIZES))
@pytest.mark.parametrize("p", [2, 3])
def test_wave_rhs_and_steps(p, size, flux):
    for nx, ny in MESHES:
        for bc in (None, ["periodic"] * 4, ["reflect", "outflow", "reflect", "reflect"]):
            announce("wave2d", p, size, flux, nx, ny, bc)
            # Butcher rows keep the smallest whole-tile meshes on this kernel too
            cfg = _cfg(nx, ny, p, size, flux=flux, integrator="bs3", **({"bc": bc} if bc else {}))
            prob, (T, R) = oracle_for(cfg)
            u = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 3)
            sol = solver_for(cfg)
            got = to_np(sol.rhs(to_dev(u)))
            sol.sync()
            assert rel_l2(got, ofr.rhs(prob, T, R, u)) < RTOL_FP64, (nx, ny)
            v = ost.limit(prob, T, R, inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 5, vacuum_frac=0.3))[0]
            ud = to_dev(v)
            w, _, _ = ostep.step(prob, v, 1e-5, (T, R))
            sol.step(ud, 1e-5)
            sol.sync()
            assert rel_l2(to_np(ud), w) < RTOL_FP64, (nx, ny)
            assert elem_max_rel(to_np(ud), w) < ELEM_RTOL, (nx, ny)


@pytest.mark.parametrize("kw", [dict(), dict(filter="exp", sensor="always", alpha=36.0)], ids=["l2", "exp_always"])
@pytest.mark.parametrize("size", list(SIZES))
@pytest.mark.parametrize("p", [2, 3])
def test_wave_ssp_steps_with_flags(p, size, kw):
    import torch
    announce("wave2d_ssp", p, size, kw)
    cfg = _cfg(5, 3, p, size, **kw)
    prob, (T, R) = oracle_for(cfg)
    v = ost.limit(prob, T, R, inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 7, vacuum_frac=0.3))[0]
    start = v.copy()
    sol = solver_for(cfg)
    ud = to_dev(v)
    dts = []
    for i in range(3):
        rec = []
        v, rdt, rfl = ostep.step(prob, v, None, (T, R), record=rec)
        dtd, fl = sol.step(ud)
        sol.sync()
        dts.append(rdt)
        assert abs(to_np(dtd)[0] / rdt - 1.0) < 1e-13, i
        check_flags(prob, T, R, to_np(fl).reshape(4, -1), rfl, rec)
        assert rel_l2(to_np(ud), v) < RTOL_FP64, i
        assert elem_max_rel(to_np(ud), v) < ELEM_RTOL, i
    u2 = to_dev(start)
    got = torch.empty(3, dtype=torch.float64, device=u2.device)
    sol.steps(u2, 3, got)
    sol.sync()
    assert np.max(np.abs(to_np(got) / np.array(dts) - 1.0)) < 1e-13
    assert rel_l2(to_np(u2), v) < RTOL_FP64


def test_static_workspace_without_room_for_the_traces():
    """60 x 25 elements, bs3: the stage arrays fit the static workspace, the face traces of this
    kernel's tiles do not; the steps then take the neighbours' traces from their states."""
    announce("wave2d_static")
    cfg = _cfg(60, 25, 3, "m15q25", integrator="bs3")
    lib = binding.load_library()
    need = ctypes.c_int64()
    P = binding.problem_from_config(cfg)
    assert lib.fr_sg_workspace_size(ctypes.byref(P), ctypes.byref(need)) == 0
    assert need.value > 64 << 20
    prob, (T, R) = oracle_for(cfg)
    u0 = project_initial(prob, cfg["ic"], (T, R))
    out = []
    for static in (False, True):
        sol = binding.Solver(cfg, static_workspace=static)
        ud = to_dev(u0)
        sol.steps(ud, 2)
        sol.sync()
        out.append(to_np(ud))
        sol.close()
    assert rel_l2(out[1], out[0]) < RTOL_FP64
