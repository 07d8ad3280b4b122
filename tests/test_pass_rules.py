"""Which lattices take multi-step passes: the rules of csrc/hlbm_pass_rules.hpp, compiled for the
host, against lattices measured with and without them on an MI355X (ratio pass / single steps):
none that a pass slows down may take it, and those that gain much must."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLAIN, WINDOW, WINDOW_REGION, ADJOINT, WINDOW_LARGE, ADJOINT_LARGE = range(6)


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2606_31707_amd", "csrc"), os.path.join(ROOT, "tests", "pass_rules_driver.cpp"),
                    "-o", exe], check=True)

    def run(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


# stencil, precision, nx, ny, nz, bc_x, bc_y, bc_z, collision, closure, kind: ratio
MEASURED_3D = {
    (1, 0, 20, 200, 50, 2, 1, 0, 1, 0.1, PLAIN): 1.74,
    (1, 1, 20, 200, 50, 2, 1, 0, 0, 0.0, PLAIN): 1.42,
    (1, 1, 10, 10, 1000, 2, 1, 0, 1, 0.1, PLAIN): 1.71,
    (1, 1, 64, 64, 64, 2, 1, 0, 0, 0.0, PLAIN): 1.30,
    (1, 1, 128, 64, 32, 2, 1, 0, 1, 0.0, PLAIN): 1.33,
    (1, 0, 64, 64, 64, 2, 1, 0, 1, 0.1, PLAIN): 1.38,
    (1, 0, 64, 20, 400, 2, 1, 0, 1, 0.0, PLAIN): 1.23,
    (1, 1, 32, 32, 32, 2, 1, 0, 1, 0.1, PLAIN): 1.17,
    (1, 1, 186, 70, 3, 0, 1, 1, 0, 0.1, PLAIN): 1.21,
    (1, 0, 9, 225, 337, 2, 0, 0, 0, 0.0, PLAIN): 2.65,
    (1, 0, 63, 75, 363, 2, 0, 0, 0, 0.1, PLAIN): 1.22,
    (1, 1, 63, 375, 145, 2, 1, 0, 0, 0.0, PLAIN): 1.22,
    (1, 1, 81, 91, 368, 2, 1, 1, 0, 0.0, PLAIN): 1.15,
    (1, 1, 64, 64, 64, 2, 1, 0, 0, 0.1, WINDOW): 1.37,
    (1, 1, 10, 10, 1000, 2, 1, 0, 0, 0.0, WINDOW): 1.35,
    (1, 0, 64, 20, 400, 2, 1, 0, 0, 0.1, WINDOW): 1.20,
    (1, 0, 34, 308, 93, 2, 0, 0, 0, 0.0, WINDOW): 1.10,
    (1, 0, 64, 20, 400, 2, 1, 0, 0, 0.1, WINDOW_REGION): 1.25,
    (1, 1, 20, 200, 50, 2, 1, 0, 0, 0.1, WINDOW_REGION): 1.37,
    (1, 1, 76, 402, 159, 2, 0, 0, 0, 0.0, WINDOW_REGION): 1.35,
    (1, 0, 63, 75, 363, 2, 0, 0, 0, 0.0, ADJOINT): 1.45,
    (1, 0, 76, 402, 159, 2, 0, 0, 0, 0.0, ADJOINT): 1.24,
    (1, 0, 63, 375, 145, 2, 1, 0, 0, 0.0, ADJOINT): 1.22,
    (1, 0, 192, 96, 64, 2, 1, 0, 0, 0.0, ADJOINT): 1.28,
    # and gains
    (1, 0, 756, 168, 84, 2, 0, 0, 0, 0.0, PLAIN): 0.70,
    (1, 0, 96, 48, 16, 2, 1, 0, 0, 0.0, PLAIN): 0.64,
    (1, 0, 16, 16, 16, 2, 1, 0, 0, 0.0, PLAIN): 0.87,
    (1, 0, 300, 128, 64, 2, 1, 0, 1, 0.1, PLAIN): 0.77,
    (1, 1, 768, 384, 128, 2, 0, 0, 0, 0.0, PLAIN): 0.77,
    (1, 1, 130, 29, 64, 0, 0, 0, 0, 0.0, PLAIN): 0.74,
    (1, 1, 696, 97, 69, 2, 1, 0, 1, 0.1, PLAIN): 0.87,
    (1, 0, 756, 168, 84, 2, 1, 0, 0, 0.0, WINDOW): 0.59,
    (1, 0, 300, 128, 64, 2, 1, 0, 0, 0.1, WINDOW): 0.60,
    (1, 1, 192, 96, 64, 2, 1, 0, 0, 0.0, WINDOW): 0.81,
    (1, 0, 16, 16, 16, 2, 1, 0, 0, 0.1, WINDOW_REGION): 0.87,
    (1, 1, 32, 32, 32, 2, 1, 0, 0, 0.0, WINDOW_REGION): 0.82,
    (1, 1, 768, 384, 128, 2, 0, 0, 0, 0.1, WINDOW_REGION): 0.97,
    (1, 0, 756, 168, 84, 2, 1, 0, 0, 0.0, ADJOINT): 0.67,
    (1, 0, 300, 128, 64, 2, 1, 0, 0, 0.1, ADJOINT): 0.79,
}


def test_3d_lattices_take_passes_where_they_pay(ask):
    for row, (_, pays) in zip(MEASURED_3D, ask(MEASURED_3D)):
        if row[10] != ADJOINT:
            assert pays == (2 if MEASURED_3D[row] < 1.0 else 1), row


def test_3d_lattices_without_a_pass_that_pays_hold_no_arrays_for_it(ask):
    narrow = (1, 1, 9, 225, 337, 2, 0, 0, 0, 0.1, PLAIN)
    assert ask([narrow])[0] == (0, 1)
    for row, (held, _) in zip(MEASURED_3D, ask(MEASURED_3D)):
        if row[10] == ADJOINT:
            assert (held > 0) == (MEASURED_3D[row] < 1.0), row


MEASURED_2D = {
    (0, 0, 7, 8990, 1, 2, 1, 0, 0, 0.0, PLAIN): 1.12,
    (0, 0, 7, 8990, 1, 2, 1, 0, 1, 0.1, PLAIN): 1.51,
    (0, 0, 19, 8747, 1, 2, 0, 0, 0, 0.1, PLAIN): 1.13,
    (0, 1, 19, 8747, 1, 2, 0, 0, 0, 0.1, PLAIN): 1.26,
    (0, 1, 7, 8990, 1, 2, 1, 0, 0, 0.1, PLAIN): 1.22,
    (0, 1, 11, 4951, 1, 2, 0, 0, 1, 0.1, PLAIN): 1.18,
    (0, 1, 289, 835, 1, 2, 1, 0, 1, 0.1, PLAIN): 1.14,
    (0, 1, 3093, 79, 1, 2, 1, 0, 1, 0.1, PLAIN): 1.12,
    (0, 2, 19, 8747, 1, 2, 0, 0, 1, 0.1, PLAIN): 1.21,
    (0, 2, 4081, 32, 1, 2, 1, 0, 0, 0.1, WINDOW): 1.17,
    (0, 2, 62, 1096, 1, 2, 0, 0, 0, 0.1, WINDOW): 1.11,
    (0, 0, 512, 256, 1, 2, 1, 0, 0, 0.1, WINDOW_LARGE): 1.19,
    (0, 0, 4081, 32, 1, 2, 1, 0, 0, 0.1, WINDOW_LARGE): 1.08,
    (0, 0, 1700, 148, 1, 2, 1, 0, 0, 0.0, ADJOINT): 1.11,
    (0, 0, 289, 835, 1, 2, 1, 0, 0, 0.1, ADJOINT_LARGE): 1.06,
    (0, 1, 1700, 148, 1, 2, 1, 0, 0, 0.0, ADJOINT_LARGE): 1.13,
    (0, 1, 556, 584, 1, 2, 0, 0, 0, 0.1, ADJOINT_LARGE): 1.09,
    (0, 1, 422, 356, 1, 2, 1, 0, 0, 0.0, ADJOINT_LARGE): 1.08,
    # and gains: the levels they take
    (0, 0, 220, 41, 1, 2, 1, 0, 0, 0.0, PLAIN): 4,
    (0, 0, 1100, 410, 1, 2, 1, 0, 1, 0.1, PLAIN): 4,
    (0, 1, 8192, 4096, 1, 2, 1, 0, 0, 0.0, PLAIN): 4,
    (0, 1, 400, 160, 1, 2, 1, 0, 0, 0.1, PLAIN): 4,
    (0, 2, 1100, 410, 1, 2, 1, 0, 0, 0.0, PLAIN): 2,
    (0, 2, 8192, 4096, 1, 2, 1, 0, 0, 0.0, PLAIN): 4,
    (0, 1, 1024, 512, 1, 2, 1, 0, 0, 0.1, WINDOW): 4,
    (0, 0, 1024, 512, 1, 2, 1, 0, 0, 0.1, WINDOW): 2,
    (0, 2, 1100, 410, 1, 2, 1, 0, 0, 0.1, WINDOW): 4,
    (0, 1, 1100, 410, 1, 2, 1, 0, 0, 0.0, WINDOW_LARGE): 2,
    (0, 0, 1100, 410, 1, 2, 1, 0, 0, 0.1, WINDOW_LARGE): 2,
    (0, 2, 8192, 4096, 1, 2, 1, 0, 0, 0.0, WINDOW_LARGE): 4,
    (0, 0, 400, 160, 1, 2, 1, 0, 0, 0.0, ADJOINT): 2,
    (0, 0, 447, 480, 1, 2, 1, 0, 0, 0.0, ADJOINT): 2,
    (0, 1, 400, 160, 1, 2, 1, 0, 0, 0.0, ADJOINT_LARGE): 2,
    (0, 1, 1024, 512, 1, 2, 1, 0, 0, 0.1, ADJOINT_LARGE): 4,
    (0, 2, 8192, 4096, 1, 2, 1, 0, 0, 0.0, ADJOINT): 4,
}


def test_2d_lattices_take_passes_where_they_pay(ask):
    for row, (held, steps) in zip(MEASURED_2D, ask(MEASURED_2D)):
        ratio = MEASURED_2D[row]
        assert steps == (ratio if ratio >= 2 else 1), row
        assert held > 0  # (whether windows have a region, and the closure, may change later)


# precision, kind, whether the group's other list takes passes, workgroups: ratio
MEASURED_PACKED = {
    (0, WINDOW, 0, 25): 1.59, (0, WINDOW, 0, 647): 1.16, (0, WINDOW, 0, 1917): 1.06, (1, WINDOW, 0, 15): 1.10,
    (2, WINDOW, 0, 13): 1.14, (1, PLAIN, 0, 74): 1.04, (2, PLAIN, 0, 63): 1.08, (0, PLAIN, 0, 54): 1.09,
    (0, ADJOINT, 0, 27): 1.31, (0, ADJOINT, 0, 276): 1.10, (1, ADJOINT, 0, 106): 1.31, (2, ADJOINT, 0, 3898): 1.24,
    (1, WINDOW, 0, 173): 0.81, (2, WINDOW, 0, 264): 0.76, (1, WINDOW, 0, 4539): 0.54, (0, PLAIN, 0, 204): 0.92,
    (0, PLAIN, 0, 776): 0.81, (1, PLAIN, 0, 1516): 0.87, (0, ADJOINT, 0, 430): 0.92, (0, ADJOINT, 0, 1934): 0.85,
    (0, WINDOW, 1, 9): 0.66, (1, ADJOINT, 1, 9): 0.60, (0, ADJOINT, 1, 5029): 0.71, (1, WINDOW, 1, 4773): 0.53,
}


def test_packed_lists_take_passes_where_they_pay(ask):
    rows = [(0, p, other, blocks, 0, 0, 0, 0, 0, 0.0, kind) for p, kind, other, blocks in MEASURED_PACKED]
    for key, (_, pays) in zip(MEASURED_PACKED, ask(rows)):
        assert pays == (MEASURED_PACKED[key] < 1.0), key


def test_plans_of_extreme_shapes_are_quick(ask):
    """A plan looks at a bounded number of chunkings however many planes there are."""
    rows = [(1, 1, 2, 1, 1 << 30, 0, 0, 0, 0, 0.0, PLAIN), (1, 0, 2, 1 << 15, 1 << 15, 0, 0, 0, 0, 0.0, PLAIN),
            (1, 1, (1 << 31) - 1, 1, 1, 0, 0, 0, 0, 0.0, PLAIN), (1, 1, 2, 1 << 30, 1, 0, 0, 0, 0, 0.0, PLAIN)]
    assert ask(rows) == [(0, 1)] * 4  # two columns fill no tile, one plane no pass
