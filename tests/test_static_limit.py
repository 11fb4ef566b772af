"""The largest meshes that fr_sg_init_static takes.  Tables and buffers that only make steps faster do
not count against the 64 MiB, so these stay where they are when a kernel gains some.  Needs no GPU:
a problem that is taken gets as far as the device."""

import ctypes
import os

import numpy as np
import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2112_05946_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2112_05946_amd import build
        build.build()
    return binding.load_library()


def _taken(lib, P):
    ctx = ctypes.c_void_p()
    st = lib.fr_sg_init_static(ctypes.byref(P), None, ctypes.byref(ctx))
    if ctx.value:
        lib.fr_sg_destroy(ctx)
    assert st in (0, -2, -3), lib.fr_sg_last_error(None).decode()
    return st != -2


def _problem(name, precision="fp64", **kw):
    from paper_2112_05946_amd import binding, inputs
    return binding.problem_from_config(dict(getattr(inputs, name), **kw), precision)


@pytest.mark.parametrize("name,kw,field,largest", [
    ("ADVECTION", dict(), "nx", 54094),
    ("BURGERS", dict(), "nx", 22540),
    ("BURGERS", dict(precision="fp32"), "nx", 22540),
    ("SOD", dict(), "nx", 8523),
    ("SOD_HLL_BS3", dict(), "nx", 6077),
    ("SOD", dict(p=7), "nx", 4598),
    ("SHOCK_VORTEX", dict(nx=2, integrator="bs3"), "ny", 716),
    ("SHOCK_VORTEX", dict(nx=2, integrator="bs3", gpc_order=2, nq1d=3), "ny", 1712),
    ("SHOCK_VORTEX", dict(nx=1, p=2, gpc_order=5, nq1d=6, integrator="bs3"), "ny", 892),
    ("SHOCK_VORTEX", dict(nx=5, p=4), "ny", 134),
])
def test_largest_quadrilateral_and_1d_meshes(lib, name, kw, field, largest):
    P = _problem(name, **kw)
    setattr(P, field, largest)
    assert _taken(lib, P)
    setattr(P, field, largest + 1)
    assert not _taken(lib, P)


@pytest.mark.parametrize("p,order,nq,integrator,largest", [
    (1, 4, 5, "ssprk3", 7631), (1, 3, 4, "bs3", 7632), (2, 1, 2, "ssprk3", 22132), (3, 2, 3, "ssprk3", 7802),
    (4, 1, 2, "bs3", 6557)])
def test_largest_triangle_meshes(lib, p, order, nq, integrator, largest):
    from paper_2112_05946_amd import binding, inputs
    for n, taken in ((largest, True), (largest + 1, False)):
        mesh = dict(xy=np.tile(np.array([[0.0, 0.0], [1.0, 0.0], [0.0, 1.0]]), (n, 1, 1)),
                    nbr=np.full((n, 3), -1, np.int32), nbr_face=np.full((n, 3), -1, np.int32))
        cfg = dict(inputs.tri_shock_vortex(4), p=p, gpc_order=order, nq1d=nq, integrator=integrator, mesh=mesh,
                   bc=["outflow"] * 4)
        assert _taken(lib, binding.problem_from_config(cfg)) == taken
