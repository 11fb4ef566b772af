"""1D meshes beyond one workgroup per compute unit: the wide windows of problems with few nodes, and
the calls for which a launch per stage is faster and which therefore take it, against the oracle.
The passes recorded by the library tell the route: whole steps are one pass beside the CFL pass."""

import pytest

from gpu_util import RTOL_FP64, announce, oracle_for, rel_l2, solver_for, to_dev, to_np
from oracle import stepper as ostep
from oracle.initial import project_initial
from paper_2112_05946_amd import inputs

pytestmark = pytest.mark.gpu


def _cfg(base, E, p, order, nq, **kw):
    return dict(inputs.small(base, E), p=p, gpc_order=order, nq1d=nq, **kw)


# (label, problem, precision, whole step in one launch)
CASES = [
    ("sod_wide", _cfg(inputs.SOD, 9000, 3, 2, 3), "fp64", True),                   # 17 elements per workgroup
    ("sod_widest", _cfg(inputs.SOD, 42001, 1, 2, 3), "fp64", True),                # 82, the last one short
    ("sod_wide_rk4", _cfg(inputs.SOD, 20011, 2, 3, 4, integrator="rk4"), "fp64", True),
    ("burgers_wide", _cfg(inputs.BURGERS, 70001, 3, 2, 3), "fp64", True),          # 68
    ("one_node", dict(_cfg(inputs.ADVECTION, 262145, 1, 0, 1)), "fp64", True),     # 250: every slot of a window
    ("burgers_12_nodes", _cfg(inputs.BURGERS, 8209, 3, 8, 12), "fp64", True),      # 15
    ("burgers_p4_24_nodes", _cfg(inputs.BURGERS, 4101, 4, 10, 24), "fp64", False),
    ("burgers_p4_32_nodes", _cfg(inputs.BURGERS, 4101, 4, 8, 32), "fp64", True),
    ("sod_rk4_few_elements", dict(_cfg(inputs.SOD, 2100, 3, 4, 5, integrator="rk4"), rdim=2), "fp64", False),
    ("sod_p4_rk4", _cfg(inputs.SOD, 1400, 4, 10, 24, integrator="rk4"), "fp64", False),
    ("sod_fp32_second_round", inputs.small(inputs.SOD, 4096), "fp32", False),
    ("sod_fp32", inputs.small(inputs.SOD, 8192), "fp32", True),
]


@pytest.mark.parametrize("label,cfg,precision,whole", CASES)
def test_large_1d_mesh(label, cfg, precision, whole):
    announce("step1d_sizes", label)
    prob, (T, R) = oracle_for(cfg)
    u = project_initial(prob, cfg["ic"], (T, R))
    sol = solver_for(cfg, precision)
    sol.timing(True)
    ud = to_dev(u)
    sol.steps(ud, 2)
    sol.sync()
    passes = sol.timing_read()
    assert (set(passes) <= {"cfl", "stage1"}) == whole, passes
    for _ in range(2):
        u, _, _ = ostep.step(prob, u, None, (T, R))
    # FP32-mixed: dt R is formed in FP32, and dt times the largest derivative weight over J is O(1)
    assert rel_l2(to_np(ud), u) < (RTOL_FP64 if precision == "fp64" else 1e-5)
