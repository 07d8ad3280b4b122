"""CPU checks of bench.py's account of multi-step passes: trace rows of their kernels, and the bytes
per update of the launches that were taken."""
import os
import sys
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_pass_kernels_map_to_sweep_kinds_and_steps():
    import bench
    cases = {
        "void hlbm::k_march2d<double, 4, false, false>(hlbm::Geo, hlbm::MarchColl)": ("primal_pass", 4),
        "_ZN4hlbm9k_march2dIDF16_Li2ELb0ELb1EEEvNS_3GeoE": ("primal_pass", 2),
        "void hlbm::k_window2d<float, 2, false, true>(hlbm::Geo)": ("primal_window_pass", 2),
        "void hlbm::k_march2d_adjoint<float, 4>(hlbm::Geo)": ("adjoint_pass", 4),
        "void hlbm::k_march3d<float, false, true>(hlbm::Geo)": ("primal_pass", 2),
        "void hlbm::(anonymous namespace)::k_march3d_adjoint<double>(hlbm::Geo)": ("adjoint_pass", 2),
        "void hlbm::k_window3d<float, true>(hlbm::Geo)": ("primal_window_pass", 2),
        "void hlbm::k_march3d_adjoint<double>(hlbm::Geo)": ("adjoint_pass", 2),
        "void hlbm::k_window_region_copy<19, float, 2>(hlbm::ObjBox)": ("region_pass", 1),
        "void hlbm::k_window_region_copy<19, float, 1>(hlbm::ObjBox)": ("region", 1),
        "void hlbm::k_primal<19, float, true, 3, false>(hlbm::Geo)": ("primal_window", 1),
        "__amd_rocclr_copyBuffer": (None, 1),
    }
    for name, (kind, steps) in cases.items():
        assert bench.kernel_kind(name)[0] == kind, name
        assert bench.kernel_steps(name) == steps, name


def test_bytes_of_the_launches_taken():
    """The LES window: a pass of two moves 152 B of populations, 4 of porosity and 80 of sums a cell
    (118 a step) and the drag plane's part, single steps 206; a run half in passes the mean."""
    import bench
    from paper_2606_31707_amd import hlbm as H
    from paper_2606_31707_amd import inputs as I
    w = I.les_re3900()
    d = H.make_desc(stencil=H.D3Q19, precision=H.FP32, nx=w.nx, ny=w.ny, nz=w.nz, tau=w.tau, cs=w.cs)
    single = {"primal": 156.0, "primal_window": 206.2, "adjoint": 172.0}

    def lattice(passes):
        return SimpleNamespace(desc=d, q=19, n=w.n, bytes_per_update=lambda: single, passes=lambda: passes)

    cells = bench.region_cells_of(w)
    assert cells == 288 * 128
    plane = (16 * 12 / 2 + 2 * 128) * cells / w.n
    G = lattice({"primal": (8, 4), "primal_window": (8, 4), "adjoint": (0, 0)})
    t = bench.taken_bytes_per_update(G, {"primal": 8, "primal_window": 16, "adjoint": 8}, None, cells)
    assert t["primal"] == (78.0, 1.0, 2.0)
    assert t["primal_window"][0] == pytest.approx(0.5 * 206.2 + 0.5 * (118.0 + plane))
    assert t["adjoint"] == (172.0, 0.0, 1.0)
    d2 = H.make_desc(precision=H.FP64, nx=1100, ny=410)
    G = SimpleNamespace(desc=d2, q=9, n=1100 * 410)
    assert bench.pass_bytes_per_update(G)["primal"](4) == (2 * 72 + 8) / 4


def test_short_kernel_names():
    import bench
    for name, want in (
            ("void hlbm::k_window3d<float, true>(hlbm::Geo, hlbm::Window)", "hlbm::k_window3d<float, true>"),
            ("void hlbm::(anonymous namespace)::k_packed2d<float>(hlbm::PackedPasses)", "hlbm::k_packed2d<float>"),
            ("__amd_rocclr_copyBuffer", "__amd_rocclr_copyBuffer")):
        assert bench.short_kernel_name(name) == want
