"""Which steps go through multi-step passes, by the library's own count: the lattices, step
counts and options of the bitwise tests (test_gpu_march.py, in the build that takes passes
everywhere) do take them, the calls that must take single steps do not, and the default build's
large and small lattices follow the rules."""
import math

import pytest

from tests import test_gpu_march as M
from tests.pairs import say

pytestmark = pytest.mark.gpu


@pytest.fixture
def everywhere(monkeypatch):
    from paper_2606_31707_amd import hlbm as H
    from paper_2606_31707_amd.build import CANARY_PATH
    monkeypatch.setattr(H, "_lib", H.open_library(CANARY_PATH))
    return H


def counts(L):
    p = L.pass_steps()
    return p["primal"], p["primal_window"], p["adjoint"]


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("bc", [(2, 1, 0), (2, 0, 0), (0, 0, 0), (0, 1, 0)])
def test_bitwise_2d_cases_take_passes(everywhere, prec, bc):
    H = everywhere
    for i, (nx, ny) in enumerate(M.SIZES_2D):
        coll, cs = ((0, 0.0), (0, 0.1), (1, 0.0), (1, 0.1))[i % 4]
        say("pass counts", prec, bc, nx, ny, coll, cs)
        L = M.lattice(H, H.D2Q9, (nx, ny, 1), prec, bc, coll, cs)
        L.run_primal(4)        # two passes of two
        assert counts(L)[0] == 4
        L.run_primal(7)        # 4, 2, one step
        assert counts(L)[0] == 4 + 6
        L.run_primal(1)        # back to an even layout
        L.run_primal(14)
        assert counts(L)[0] == 10 + 14
        L.run_primal(2)        # no pair of passes
        assert counts(L)[0] == 24
        L.close()
        for obj in ("ffa", "diss"):
            L = M.lattice(H, H.D2Q9, (nx, ny, 1), prec, bc, 0, cs)
            lo, hi = M.REGIONS_2D[obj](nx, ny)
            L.set_objective(H.OBJ_FFA if obj == "ffa" else H.OBJ_DISS, lo, hi, u0=0.04)
            L.run_primal(9, accumulate=True)
            # (tiny lattices' pending slots do not hold a region's records)
            assert counts(L)[1] == 8 or (prec != 0 and nx * ny < 1000)
            L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_FROZEN, max_iters=14)
            assert counts(L) == (0, counts(L)[1], 14)
            L.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("bc", [(2, 0, 0), (2, 1, 1), (0, 0, 0)])
def test_bitwise_3d_cases_take_passes(everywhere, prec, bc):
    H = everywhere
    for i, size in enumerate(M.SIZES_3D):
        coll, cs = ((0, 0.0), (0, 0.1), (1, 0.0), (1, 0.1))[i % 4]
        say("pass counts", prec, bc, size, coll, cs)
        L = M.lattice(H, H.D3Q19, size, prec, bc, coll, cs)
        L.run_primal(6)
        assert counts(L)[0] == 4   # a pair of passes, two steps
        L.close()
        L = M.lattice(H, H.D3Q19, size, prec, bc, 0, cs)
        L.run_primal(8, accumulate=True)
        assert counts(L)[1] == 8
        L.set_objective(H.OBJ_DISS, (1, 0, 0), (size[0] - 2, size[1] - 1, size[2] - 1), u0=0.04)
        L.run_primal(8, accumulate=True)
        L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_FROZEN, max_iters=8)
        region = (size[0] - 2) * size[1] * size[2]
        large = region * 8 > L.n  # its terms do not fit beside two levels
        assert counts(L)[1] == (8 if large else 16) or prec != 0
        assert counts(L)[2] == (8 if prec == 0 else 0)
        L.close()


def test_calls_that_take_single_steps(everywhere):
    """Body force, walls on x, FP16S in 3D, J_MEA and HRR windows, tracked populations, the
    differentiated closure, a limit of no optional arrays, a run on an odd layout, a capture."""
    import torch
    H = everywhere
    say("pass counts: single steps")
    kw = dict(stencil=H.D2Q9, nx=96, ny=40, tau=0.6, u_in=0.04)
    for more in (dict(force=(1e-7, 0.0, 0.0), bc_x=0), dict(bc_x=1), dict(optional_limit=0),
                 dict(stencil=H.D3Q19, precision=H.FP16S, nz=8)):
        L = H.Lattice(**{**kw, **more})
        L.run_primal(16)
        L.run_primal(16, accumulate=True)
        assert counts(L)[:2] == (0, 0), more
        L.close()
    for more in (dict(collision=H.COLL_HRR), dict(track_mean_populations=True)):
        L = H.Lattice(**{**kw, **more})
        L.run_primal(16)
        L.run_primal(16, accumulate=True)
        assert counts(L)[:2] == (16, 0), more
        L.close()
    L = H.Lattice(cs=0.1, track_mean_populations=True, **kw)
    L.build_cylinder(24.0, 19.5, 10.0)
    L.set_objective(H.OBJ_MEA, (10, 5, 0), (40, 35, 0), u0=math.pi * 10.0)
    L.run_primal(16, accumulate=True)
    L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_FROZEN, max_iters=8)
    L.set_objective(H.OBJ_FFA, (60, 0, 0), (60, 39, 0), u0=0.04)
    L.run_primal(16, accumulate=True)
    L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_DIFFERENTIATED, max_iters=8)
    assert counts(L) == (0, 0, 0)
    L.run_primal(1)
    L.run_primal(16)  # one step to an even layout, passes, one step
    assert counts(L)[0] == 14
    L.close()
    stream = torch.cuda.Stream()
    L = H.Lattice(stream=stream.cuda_stream, **kw)
    L.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        L.run_primal(16)
    assert counts(L)[0] == 0
    L.close()


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_packed_members_take_passes(everywhere, prec):
    H = everywhere
    say("pass counts: packed", prec)
    members = M._members(H, prec)
    before = [counts(L) for L, _ in members]
    g = H.Group()
    g.set([L for L, _ in members], [mode for _, mode in members])
    g.step(21)
    g.synchronize()
    for (L, mode), b in zip(members, before):
        assert counts(L)[mode] - b[mode] == 20, mode
    g.close()
    for L, _ in members:
        L.close()


def test_the_default_build_follows_the_rules():
    from paper_2606_31707_amd import hlbm as H
    say("pass counts: rules")
    for kw, steps in ((dict(nx=220, ny=41, precision=H.FP64), 16), (dict(nx=7, ny=8990, precision=H.FP64, cs=0.1), 0),
                      (dict(stencil=H.D3Q19, nx=96, ny=48, nz=16, precision=H.FP64), 16),
                      (dict(stencil=H.D3Q19, nx=20, ny=200, nz=50, precision=H.FP32), 0)):
        L = H.Lattice(tau=0.6, u_in=0.04, **kw)
        L.run_primal(16)
        assert counts(L)[0] == steps, kw
        L.close()
    kw = dict(precision=H.FP64, tau=0.6, u_in=0.04)
    for sizes, mode, steps in (([(96, 48)] * 2, H.GROUP_PRIMAL_WINDOW, 0), ([(512, 256)] * 3, H.GROUP_PRIMAL, 20),
                               ([(96, 48)] * 2, H.GROUP_PRIMAL, 0)):
        lats = [H.Lattice(nx=nx, ny=ny, **kw) for nx, ny in sizes]
        g = H.Group()
        g.set(lats, [mode] * len(lats))
        g.step(21)
        g.synchronize()
        assert all(counts(L)[mode] == steps for L in lats), sizes
        g.close()
        for L in lats:
            L.close()
