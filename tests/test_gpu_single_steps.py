"""Single steps again: tests of the streaming sweeps, the grouped window sums, the region pass and
the other tile shape whose lattices now take multi-step passes, on lattices without the arrays for
them."""
import numpy as np
import pytest

from tests import test_gpu_march as M
from tests.pairs import say
from tests.test_gpu_cache_policy import (  # noqa: F401 (collected here too)
    test_above_threshold_full_query, test_lattice_above_the_threshold, test_policies_give_identical_results,
    test_policies_identical_d3q19_les, test_policies_identical_hrr, test_policies_identical_region_pass_and_mea,
    test_streaming_sweep_matches_oracle)
from tests.test_gpu_footprint import test_device_bytes_equal_the_footprint  # noqa: F401
from tests.test_gpu_grouped_window import test_grouped_sums_equal_ungrouped_launches  # noqa: F401
from tests.test_gpu_race_canary import test_other_tile_shape_and_order_give_the_same_results  # noqa: F401
from tests.test_gpu_window_region import test_window_mean_and_mean_flow_adjoint  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def without_optional_arrays(monkeypatch):
    from paper_2606_31707_amd import hlbm as H

    class Single(H.Lattice):
        made = []

        def __init__(self, *args, **kw):
            kw = {"optional_limit": 0, **kw}
            super().__init__(*args, **kw)
            self.single = kw["optional_limit"] == 0
            self.made.append(self)

        def close(self):
            if getattr(self, "_h", None) is not None and self.single:
                assert not any(self.pass_steps().values())
            super().close()

        def __del__(self):
            super().close()

    monkeypatch.setattr(H, "Lattice", Single)
    yield
    for lat in Single.made:  # closed ones have passed
        lat.close()


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("stencil", [0, 1])
def test_passes_equal_streaming_single_steps(stencil, prec, monkeypatch):
    """Lattices larger than the caches: single steps under the automatic (streaming) policy against
    the same steps in passes, where there are passes."""
    from paper_2606_31707_amd import hlbm as H
    say("streaming singles", stencil, prec)
    size = ((2803, 1501, 1), (4001, 1803, 1), (4507, 2709, 1))[prec] if stencil == 0 else \
        ((310, 96, 64), (181, 157, 129), (256, 190, 141))[prec]
    outs = []
    for limit in (0, None):
        L = M.lattice(H, stencil, size, prec, (2, 1, 0), 0, 0.1, optional_limit=limit)
        x = size[0] // 2
        L.set_objective(H.OBJ_FFA, (x, 0, 0), (x, size[1] - 1, size[2] - 1), u0=0.04)
        L.run_primal(9)
        L.run_primal(1)
        L.run_primal(9, accumulate=True)
        L.solve_adjoint(H.SOURCE_MEAN, tau_adj=0.6, turb=H.TURB_FROZEN, max_iters=6)
        if limit is None and not (stencil == 1 and prec == 2):
            p = L.pass_steps()
            assert p["primal"] == 8 and p["primal_window"] == 8, p
            assert p["adjoint"] == (0 if stencil == 1 and prec == 1 else (4 if stencil == 1 else 6)), p
        outs.append((L.field(H.FIELD_U), L.field(H.FIELD_MEAN_U), L.objective(1), L.gradient()))
        L.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
