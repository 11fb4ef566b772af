"""The FP64 2D stage kernels at both sides of the rule that chooses between them: the pair kernel (4 x 2
element tiles) on whole and cut tiles, p = 2 and p = 3, at every mode count, from one workgroup more
than the wave kernel takes; the wave kernel's walk in blocks of 8 x 8 tiles; and the matrix-core
right-hand side of small meshes of 10 modes.  Long strips of elements keep the oracle's work small.
Which kernel serves a mesh shows in the size of its face-trace buffers."""

import ctypes

import numpy as np
import pytest

from gpu_util import ELEM_RTOL, RTOL_FP64, announce, elem_max_rel, oracle_for, rel_l2, solver_for, to_dev, to_np
from oracle import fr as ofr
from oracle import stabilize as ost
from oracle import stepper as ostep
from paper_2112_05946_amd import binding, inputs

pytestmark = pytest.mark.gpu

SIZES = {"m15q25": (4, 5, 2), "m10q16": (3, 4, 2), "m6q9": (2, 3, 2), "m3q4": (2, 4, 1)}


def _cfg(nx, ny, p, size, **kw):
    order, nq, rdim = SIZES[size]
    return dict(inputs.small(inputs.SHOCK_VORTEX, nx, ny), p=p, gpc_order=order, nq1d=nq, rdim=rdim, **kw)


def _trace_faces(cfg):
    """Element faces in a face-trace buffer of the problem: the workspace beyond that of one element."""
    lib = binding.load_library()
    modes = {"4": 15, "3": 10, "2": 6}[str(cfg["gpc_order"])] if cfg["rdim"] == 2 else cfg["gpc_order"] + 1
    align = lambda n: (n + 255) // 256 * 256
    face = 8 * 4 * (cfg["p"] + 1) * modes

    def rest(nx, ny):
        P = binding.problem_from_config(dict(cfg, nx=nx, ny=ny, integrator="ssprk3"))
        n = ctypes.c_int64()
        assert lib.fr_sg_workspace_size(ctypes.byref(P), ctypes.byref(n)) == 0
        return n.value - 2 * align(8 * 4 * modes * nx * ny * (cfg["p"] + 1) ** 2)
    one = 2 * align(8 * face)  # the wave kernel's 2 x 2 tile
    return round(((rest(cfg["nx"], cfg["ny"]) - rest(1, 1) + one) // 2) / face)


def _pair_faces(nx, ny):
    return ((nx + 3) // 4) * ((ny + 1) // 2) * 12


def _wave_faces(nx, ny):
    return ((nx + 1) // 2) * ((ny + 1) // 2) * 8


# 257 workgroups of the pair kernel (145 with 9 nodes): one column, cut tiles, whole tiles
PAIR = [("m15q25", 1, 514, 2), ("m15q25", 1, 513, 3), ("m10q16", 1, 514, 2), ("m10q16", 5, 258, 3), ("m10q16", 4, 514, 3),
        ("m6q9", 5, 146, 2), ("m6q9", 3, 290, 3), ("m6q9", 4, 290, 3), ("m3q4", 2, 513, 2), ("m3q4", 1, 514, 3),
        ("m3q4", 4, 514, 3)]
# the last mesh that the wave kernel takes, and meshes of 8 x 8 of its tiles
WAVE = [("m10q16", 1, 512, 3), ("m6q9", 5, 144, 2), ("m6q9", 1, 288, 3), ("m3q4", 1, 512, 2), ("m15q25", 16, 16, 3),
        ("m10q16", 15, 16, 2)]


@pytest.mark.parametrize("integrator", ["ssprk3", "bs3"])
@pytest.mark.parametrize("kernel,size,nx,ny,p", [("pair",) + c for c in PAIR] + [("wave",) + c for c in WAVE])
def test_both_sides_of_the_rule(kernel, size, nx, ny, p, integrator):
    announce("stage2d_rules", kernel, size, nx, ny, p, integrator)
    cfg = _cfg(nx, ny, p, size, integrator=integrator, flux="hll" if p == 2 else "rusanov")
    assert _trace_faces(cfg) == (_pair_faces if kernel == "pair" else _wave_faces)(nx, ny)
    prob, (T, R) = oracle_for(cfg)
    u = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 3)
    sol = solver_for(cfg)
    got = to_np(sol.rhs(to_dev(u)))
    sol.sync()
    assert rel_l2(got, ofr.rhs(prob, T, R, u)) < RTOL_FP64
    # two steps of one call: traces and CFL maximum handed on, the limiter acting.  Among a thousand
    # elements near vacuum some answer a rounding of the state with 1e-11 of themselves: the bars
    # are widened by ten times what the oracle itself makes of one
    v = ost.limit(prob, T, R, inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 5, vacuum_frac=0.3))[0]
    w = v * (1.0 + 2.2e-16 * np.random.default_rng(0).choice([-1, 0, 1], size=v.shape))
    ud = to_dev(v)
    sol.steps(ud, 2)
    sol.sync()
    for _ in range(2):
        v, _, _ = ostep.step(prob, v, None, (T, R))
        w, _, _ = ostep.step(prob, w, None, (T, R))
    assert rel_l2(to_np(ud), v) < RTOL_FP64 + 10 * rel_l2(w, v)
    assert elem_max_rel(to_np(ud), v) < ELEM_RTOL + 10 * elem_max_rel(w, v)


@pytest.mark.parametrize("flux", ["rusanov", "hll"])
@pytest.mark.parametrize("nx,ny,matrix_cores", [(2, 2, True), (6, 4, True), (8, 4, True), (4, 288, True), (4, 290, False),
                                                (5, 4, False)])
def test_right_hand_side_of_10_modes(nx, ny, matrix_cores, flux):
    announce("rhs_10_modes", nx, ny, flux)
    cfg = _cfg(nx, ny, 3, "m10q16", flux=flux)
    prob, (T, R) = oracle_for(cfg)
    u = inputs.fuzz_euler(2, R.M, prob.E, prob.nsp, 4)
    sol = solver_for(cfg)
    sol.timing(True)
    got = to_np(sol.rhs(to_dev(u)))
    sol.sync()
    assert ("traces" in sol.timing_read()) == matrix_cores
    assert rel_l2(got, ofr.rhs(prob, T, R, u)) < RTOL_FP64
