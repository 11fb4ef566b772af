"""The fused triangle stage kernel where its split can go wrong: fewer triangles than a block
of four holds, one past a block, past the eighth block (blocks are dealt to eight dies), every
degree and every (modes, nodes) pair of its set (node counts that are and are not multiples
of the group of four), all boundary kinds; the right-hand side, steps with the filter and the
limiter acting from near vacuum, and chained steps, against the oracle at the FP64 parity bar."""

import numpy as np
import pytest

from gpu_util import ELEM_RTOL, RTOL_FP64, announce, check_flags, elem_max_rel, rel_l2, solver_for, to_dev, to_np
from oracle import stabilize as ost
from oracle import stepper as ostep
from oracle import tri as otri
from oracle.problem import Problem
from oracle.tables import build_tables
from paper_2112_05946_amd import inputs

pytestmark = pytest.mark.gpu

# (gpc_order, nq1d, rdim) of the (modes, nodes) pairs (15, 25), (10, 16), (6, 9), (5, 5), (3, 4)
PAIRS = {(15, 25): (4, 5, 2), (10, 16): (3, 4, 2), (6, 9): (2, 3, 2), (5, 5): (4, 5, 1), (3, 4): (2, 4, 1)}


def _cfg(n, m, p, pair, flux="rusanov", bounded=True, **kw):
    gpc, nq, rdim = PAIRS[pair]
    mesh = inputs.tri_mesh_rectangle(n, m, periodic=(not bounded,) * 2, perturb=0.2, seed=5)
    st = inputs._cons2d(*[np.array(v) for v in (1.0, 1.302, 0.0, 1.0)])
    return dict(dict(name="tri_blocks", equation="euler2d", ic="tri_vortex", element="tri", mesh=mesh, nx=1, ny=1, p=p,
                     gpc_order=gpc, nq1d=nq, rdim=rdim,
                     bc=["dirichlet", "outflow", "reflect", "reflect"] if bounded else ["outflow"] * 4,
                     bc_state=[[float(v) for v in st]] + [[0.0] * 4] * 3, gamma=inputs.GAMMA, flux=flux,
                     integrator="ssprk3", filter="none", limiter=False, cfl=0.3), **kw)


@pytest.mark.parametrize("pair", list(PAIRS))
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_rhs_over_block_remainders(p, pair):
    for n, m, flux, bounded in [(1, 1, "hll", True), (3, 1, "rusanov", True), (5, 1, "hll", True), (3, 3, "rusanov", False),
                                (17, 1, "rusanov", True)]:
        announce("tri_blocks_rhs", p, pair, n, m, flux)
        cfg = _cfg(n, m, p, pair, flux, bounded)
        prob = Problem.from_config(cfg)
        T, R = build_tables(prob)
        assert (R.M, R.Nq) == pair
        u = inputs.fuzz_euler(2, R.M, prob.E, T.n, seed=17)
        sol = solver_for(cfg)
        got = to_np(sol.rhs(to_dev(u)))
        sol.sync()
        assert rel_l2(got, otri.rhs_tri(prob, T, R, u)) < RTOL_FP64, (n, m)


@pytest.mark.parametrize("pair", [(15, 25), (10, 16), (6, 9)])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_steps_from_near_vacuum(p, pair):
    announce("tri_blocks_steps", p, pair)
    cfg = _cfg(5, 3, p, pair, limiter=True, filter="exp", sensor="always", alpha=36.0, s=8.0)
    prob = Problem.from_config(cfg)
    T, R = build_tables(prob)
    u = inputs.fuzz_euler(2, R.M, prob.E, T.n, seed=23, vacuum_frac=0.3)
    u, _ = ost.limit(prob, T, R, u)
    start = u.copy()
    sol = solver_for(cfg)
    ud = to_dev(u)
    dts = []
    for i in range(3):
        rec = []
        u, rdt, rfl = ostep.step(prob, u, None, (T, R), record=rec)
        dtd, fl = sol.step(ud)
        sol.sync()
        dts.append(rdt)
        assert abs(to_np(dtd)[0] / rdt - 1.0) < 1e-13, i
        check_flags(prob, T, R, to_np(fl).reshape(4, -1), rfl, rec)
        assert rel_l2(to_np(ud), u) < RTOL_FP64, i
        assert elem_max_rel(to_np(ud), u) < ELEM_RTOL, i
    import torch
    u2 = to_dev(start)
    got = torch.empty(3, dtype=torch.float64, device=u2.device)
    sol.steps(u2, 3, got)
    sol.sync()
    assert np.max(np.abs(to_np(got) / np.array(dts) - 1.0)) < 1e-13
    assert rel_l2(to_np(u2), u) < RTOL_FP64
