"""The fused 2D stage kernel on meshes that its 4 x 2 element tiles do not divide and on
p = 2 elements (3 x 3 points in a 4 x 4 lane row): right-hand side, steps with the
limiter acting, chained against single steps, and the element-wise pass, against the
oracle at the FP64 parity bar."""

import numpy as np
import pytest

from gpu_util import (ELEM_RTOL, RTOL_FP64, announce, check_flags, elem_max_rel, oracle_for, rel_l2, solver_for, to_dev,
                      to_np)
from oracle import fr as ofr
from oracle import stabilize as ost
from oracle import stepper as ostep
from oracle.initial import project_initial
from paper_2112_05946_amd import inputs

pytestmark = pytest.mark.gpu

PERIODIC = ["periodic"] * 4
# one element, one short of and one past a tile in either direction, several tiles
MESHES = [(1, 1), (3, 1), (4, 3), (5, 2), (2, 5), (9, 4), (7, 3), (8, 2)]


def _cfg(nx, ny, p, order=2, **kw):
    return dict(inputs.small(inputs.SHOCK_VORTEX, nx, ny), p=p, gpc_order=order, nq1d=order + 1, **kw)


def _vacuum(cfg, seed):
    prob, (T, R) = oracle_for(cfg)
    u = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, seed, vacuum_frac=0.3)
    return ost.limit(prob, T, R, u)


@pytest.mark.parametrize("bc", [None, PERIODIC], ids=["domain", "periodic"])
@pytest.mark.parametrize("p", [2, 3])
@pytest.mark.parametrize("nx,ny", MESHES)
def test_ragged_rhs_and_steps(nx, ny, p, bc):
    announce("quad_ragged", nx, ny, p, bc)
    cfg = _cfg(nx, ny, p, **({"bc": bc} if bc else {}))
    prob, (T, R) = oracle_for(cfg)
    u = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 3)
    sol = solver_for(cfg)
    got = to_np(sol.rhs(to_dev(u)))
    sol.sync()
    assert rel_l2(got, ofr.rhs(prob, T, R, u)) < RTOL_FP64
    v, _ = _vacuum(cfg, 5)
    ud = to_dev(v)
    for i in range(2):
        rec = []
        v, _, rfl = ostep.step(prob, v, 1e-5, (T, R), record=rec)
        _, fl = sol.step(ud, 1e-5)
        sol.sync()
        check_flags(prob, T, R, to_np(fl).reshape(4, -1), rfl, rec)
        assert rel_l2(to_np(ud), v) < RTOL_FP64, i
        assert elem_max_rel(to_np(ud), v) < ELEM_RTOL, i


@pytest.mark.parametrize("label,kw", [("order4", dict(order=4)), ("order3_hll_exp", dict(order=3, flux="hll", filter="exp",
                                                                                         sensor="always", alpha=36.0)),
                                      ("order2_bs3", dict(order=2, integrator="bs3")),
                                      ("order4_rdim1", dict(order=4, rdim=1))])
@pytest.mark.parametrize("p", [2, 3])
def test_ragged_chained_steps(label, kw, p):
    """Steps of one call (face traces and CFL maximum handed on) against the oracle, and the
    limiter pass, on a 7 x 5 mesh with the domain's own boundaries."""
    import torch
    announce("quad_ragged_chained", label, p)
    cfg = _cfg(7, 5, p, **kw)
    prob, (T, R) = oracle_for(cfg)
    v = project_initial(prob, cfg["ic"], (T, R))
    sol = solver_for(cfg)
    ud = to_dev(v)
    n = 3
    dts = torch.empty(n, dtype=torch.float64, device=ud.device)
    sol.steps(ud, n, dts)
    sol.sync()
    for i in range(n):
        v, rdt, _ = ostep.step(prob, v, None, (T, R))
        assert abs(float(to_np(dts)[i]) / rdt - 1.0) < 1e-13
    assert rel_l2(to_np(ud), v) < RTOL_FP64
    w = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 9, vacuum_frac=0.3)
    ref, rfl = ost.limit(prob, T, R, w)
    wd = to_dev(w)
    flags = torch.empty(prob.E, dtype=torch.uint8, device=wd.device)
    sol.limit(wd, flags)
    sol.sync()
    assert rfl.any() and np.array_equal(to_np(flags).astype(bool), rfl)
    assert elem_max_rel(to_np(wd), ref) < ELEM_RTOL
