"""The multi-step passes on every lattice that can take them, in the build without the rules that
leave small or badly divided lattices to single steps (libhlbm_canary.so): the tests of
test_gpu_march.py again, which so reach the 3D passes on a few cells and passes of four adjoint
iterations and of four FP16 steps at the edges of strips and chunks, and 3D adjoint passes on
small lattices."""
import numpy as np
import pytest

from tests import test_gpu_march as M
from tests.pairs import say
from tests.test_gpu_march import (  # noqa: F401 (collected here too)
    test_adjoint_passes_equal_single_iterations_2d, test_captured_steps_replay_between_runs_with_passes,
    test_packed_passes_equal_packed_single_steps, test_primal_passes_equal_single_steps_2d,
    test_primal_passes_equal_single_steps_3d, test_window_passes_equal_single_steps)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def every_lattice_takes_passes(monkeypatch):
    from paper_2606_31707_amd import hlbm as H
    from paper_2606_31707_amd.build import CANARY_PATH
    monkeypatch.setattr(H, "_lib", H.open_library(CANARY_PATH))


@pytest.mark.parametrize("bc", [(2, 0, 0), (2, 1, 0), (2, 1, 1), (0, 0, 0), (0, 1, 1), (2, 0, 1)])
@pytest.mark.parametrize("obj", ["ffa", "diss"])
def test_adjoint_passes_equal_single_iterations_3d_small(bc, obj):
    from paper_2606_31707_amd import hlbm as H
    for size in M.SIZES_3D:
        nx, ny, nz = size
        (lx, ly, _), (hx, hy, _) = M.REGIONS_2D[obj](nx, ny)
        say("forced adjoint passes", size, bc, obj)
        a, b = (M.lattice(H, H.D3Q19, size, 0, bc, 0, 0.1 if obj == "ffa" else 0.0) for _ in range(2))
        for L in (a, b):
            L.set_objective(H.OBJ_FFA if obj == "ffa" else H.OBJ_DISS, (lx, ly, nz // 3), (hx, hy, nz - 1), u0=0.04)
            L.run_primal(4, accumulate=True)
        M._adjoints(H, a, b, H.SOURCE_MEAN, 4, 0)
        M._adjoints(H, a, b, H.SOURCE_MEAN, 6, 4)
        assert np.array_equal(a.adjoint(), b.adjoint())
        assert np.array_equal(a.gradient(), b.gradient())
        a.close()
        b.close()
