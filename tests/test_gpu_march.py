"""Multi-step passes (several steps in one pass over memory) against the same
number of single steps: bitwise the same populations and probe record.  Sizes
at the edges of the strips (64 - 2 (K - 1) columns: 62 and 58) and row chunks,
channels narrower than one strip, every kind of end and wall the passes take,
step counts with every remainder, runs that start on an odd step."""
import numpy as np
import pytest

from tests.pairs import say

pytestmark = pytest.mark.gpu


def lattice(H, stencil, size, prec, bc, coll, cs, seed=1, **kw):
    nx, ny, nz = size
    G = H.Lattice(stencil=stencil, precision=prec, nx=nx, ny=ny, nz=nz, tau=0.56, cs=cs, bc_x=bc[0], bc_y=bc[1],
                  bc_z=bc[2], inlet_profile=H.INLET_PARABOLIC, u_in=0.04, collision=coll, **kw)
    rng = np.random.default_rng(seed)
    G.set_porosity(rng.uniform(0.0, 1.0, G.n))
    u = 0.02 * rng.uniform(-1.0, 1.0, (3, G.n))
    if stencil == H.D2Q9:
        u[2] = 0.0
    G.init_equilibrium(1.0, u)
    return G


SIZES_2D = [(3, 2), (58, 8), (59, 9), (62, 13), (63, 5), (117, 16), (130, 3), (233, 41)]


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("bc", [(2, 1, 0), (2, 0, 0), (0, 0, 0), (0, 1, 0), (1, 1, 0)])
def test_primal_passes_equal_single_steps_2d(prec, bc):
    from paper_2606_31707_amd import hlbm as H
    for i, (nx, ny) in enumerate(SIZES_2D + ([(2, 3)] if bc[0] != 2 else [])):
        coll, cs = ((0, 0.0), (0, 0.1), (1, 0.0), (1, 0.1))[i % 4]
        say("primal passes", prec, bc, nx, ny, coll, cs)
        a, b = (lattice(H, H.D2Q9, (nx, ny, 1), prec, bc, coll, cs) for _ in range(2))
        for L in (a, b):
            L.set_probe(min(nx - 1, nx // 2 + 1), ny // 2)
        for steps in (4, 7, 9, 2, 14):
            a.run_primal(steps)
            for _ in range(steps):
                b.run_primal(1)
            assert np.array_equal(a.populations(), b.populations()), (nx, ny, steps)
            assert np.array_equal(a.probe(), b.probe()), (nx, ny, steps)
        a.close()
        b.close()


REGIONS_2D = {"ffa": lambda nx, ny: ((min(nx - 2, 60), 0, 0), (min(nx - 2, 60), ny - 1, 0)),
              "diss": lambda nx, ny: ((1, ny // 5, 0), (nx - 2, ny - 1, 0))}


def _adjoints(H, a, b, source, iters, singles):
    """Runs `iters` iterations on a by its own launches and on b by single packed iterations."""
    if singles == 0:
        for L in (a, b):
            L.solve_adjoint(source, tau_adj=0.6, turb=H.TURB_FROZEN, max_iters=0)
    g = H.Group()
    g.set([b], [H.GROUP_ADJOINT])
    for _ in range(iters):
        g.step(1)
    g.synchronize()
    g.close()
    a.solve_adjoint(source, tau_adj=0.6, turb=H.TURB_FROZEN, max_iters=iters, restart=False)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("bc", [(2, 1, 0), (2, 0, 0), (0, 0, 0), (0, 1, 0)])
def test_adjoint_passes_equal_single_iterations_2d(prec, bc):
    from paper_2606_31707_amd import hlbm as H
    for i, (nx, ny) in enumerate(SIZES_2D):
        cs = (0.0, 0.1)[i % 2]
        for obj in ("ffa", "diss"):
            lo, hi = REGIONS_2D[obj](nx, ny)
            say("adjoint passes", prec, bc, nx, ny, cs, obj)
            a, b = (lattice(H, H.D2Q9, (nx, ny, 1), prec, bc, 0, cs) for _ in range(2))
            for L in (a, b):
                L.set_objective(H.OBJ_FFA if obj == "ffa" else H.OBJ_DISS, lo, hi, u0=0.04)
                L.run_primal(3)
                L.run_primal(5, accumulate=True)
            done = 0
            for iters in (4, 6, 2, 14):
                _adjoints(H, a, b, H.SOURCE_MEAN, iters, done)
                done += iters
                assert np.array_equal(a.adjoint(), b.adjoint()), (nx, ny, obj, done)
                assert np.array_equal(a.gradient(), b.gradient()), (nx, ny, obj, done)
            a.close()
            b.close()


SIZES_3D = [(3, 2, 2), (62, 14, 5), (63, 15, 4), (64, 6, 3), (130, 29, 9), (20, 7, 12)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("bc", [(2, 0, 0), (2, 1, 0), (2, 1, 1), (0, 0, 0), (0, 1, 1), (2, 0, 1)])
def test_primal_passes_equal_single_steps_3d(prec, bc):
    from paper_2606_31707_amd import hlbm as H
    for i, size in enumerate(SIZES_3D + ([(2, 3, 2)] if bc[0] != 2 else [])):
        coll, cs = ((0, 0.0), (0, 0.1), (1, 0.0), (1, 0.1))[i % 4]
        say("primal passes", prec, bc, size, coll, cs)
        a, b = (lattice(H, H.D3Q19, size, prec, bc, coll, cs) for _ in range(2))
        for L in (a, b):
            L.set_probe(min(size[0] - 1, size[0] // 2 + 1), size[1] // 2, size[2] // 2)
        for steps in (4, 7, 5, 2):
            a.run_primal(steps)
            for _ in range(steps):
                b.run_primal(1)
            assert np.array_equal(a.populations(), b.populations()), (size, steps)
            assert np.array_equal(a.probe(), b.probe()), (size, steps)
        a.close()
        b.close()


# A small region (its terms through records), a large one (terms in the sweep; single steps in 3D),
# none.
def regions(size):
    nx, ny, nz = size
    x = min(nx - 2, 60)
    return [None, ("ffa", (x, 0, 0), (x, max(0, ny // 2 - 1), nz - 1)), ("diss", (1, ny // 5, 0), (nx - 2, ny - 1, nz - 1)),
            ("diss", (x, ny // 2, nz // 2), (min(nx - 1, x + 3), ny // 2, nz // 2))]


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("dim,bc", [(2, (2, 1, 0)), (2, (2, 0, 0)), (2, (0, 0, 0)), (2, (0, 1, 0)), (3, (2, 0, 0)),
                                    (3, (2, 1, 0)), (3, (0, 1, 1))])
def test_window_passes_equal_single_steps(dim, prec, bc):
    """Sums, objective means, probe and state of window passes, bitwise against single steps; runs
    whose remainder steps leave pending values, and a plain run before an odd start."""
    from paper_2606_31707_amd import hlbm as H
    kinds = {"ffa": H.OBJ_FFA, "diss": H.OBJ_DISS}
    sizes = [(63, 5, 1), (117, 16, 1), (130, 30, 1), (233, 41, 1)] if dim == 2 else [(63, 15, 4), (130, 29, 9), (20, 7, 12)]
    for i, size in enumerate(sizes):
        for j, region in enumerate(regions(size)):
            cs = (0.0, 0.1)[(i + j) % 2]
            say("window passes", dim, prec, bc, size, cs, region)
            a, b = (lattice(H, H.D2Q9 if dim == 2 else H.D3Q19, size, prec, bc, 0, cs) for _ in range(2))
            for L in (a, b):
                L.set_probe(min(size[0] - 1, size[0] // 2 + 1), size[1] // 2, size[2] // 2)
                if region:
                    L.set_objective(kinds[region[0]], region[1], region[2], u0=0.04)
            for steps, accumulate in ((9, True), (3, False), (8, True), (2, True)):
                a.run_primal(steps, accumulate=accumulate)
                for _ in range(steps):
                    b.run_primal(1, accumulate=accumulate)
                assert np.array_equal(a.populations(), b.populations()), (size, region, steps)
                assert np.array_equal(a.probe(), b.probe()), (size, region, steps)
            for f in [H.FIELD_MEAN_RHO, H.FIELD_MEAN_U] + ([H.FIELD_MEAN_TAU] if cs > 0 else []):
                assert np.array_equal(a.field(f), b.field(f)), (size, region, f)
            if region:
                assert a.objective(1) == b.objective(1), (size, region)
                grads = []
                for L in (a, b):
                    L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_FROZEN, max_iters=4)
                    grads.append(L.gradient())
                assert np.array_equal(*grads), (size, region)
            a.close()
            b.close()


@pytest.mark.parametrize("prec,size,cs", [(1, (4099, 1700, 1), 0.1), (2, (5003, 2500, 1), 0.0)])
def test_window_passes_with_a_large_region_beyond_the_caches(prec, size, cs):
    """Four steps a pass with the region's terms in the sweep (lattices larger than the caches)."""
    from paper_2606_31707_amd import hlbm as H
    say("large window passes", prec, size, cs)
    out = []
    for single in (False, True):
        L = lattice(H, H.D2Q9, size, prec, (2, 1, 0), 0, cs)
        L.set_objective(H.OBJ_DISS, (1, size[1] // 5, 0), (size[0] - 2, size[1] - 1, 0), u0=0.04)
        for _ in range(9 if single else 1):
            L.run_primal(1 if single else 9, accumulate=True)
        L.solve_adjoint(H.SOURCE_MEAN, turb=H.TURB_FROZEN, max_iters=2)
        out.append((L.objective(1), L.field(H.FIELD_MEAN_U), L.field(H.FIELD_U), L.gradient()))
        L.close()
    assert out[0][0] == out[1][0]
    for a, b in zip(out[0][1:], out[1][1:]):
        assert np.array_equal(a, b)


# FP64 lattices just beyond the caches: rows and planes beside walls in and next to a tile's halo.
@pytest.mark.parametrize("size,bc,obj", [((124, 121, 113), (2, 0, 0), "ffa"), ((125, 121, 113), (2, 1, 1), "diss"),
                                         ((190, 94, 97), (2, 0, 1), "diss"), ((61, 127, 221), (2, 1, 0), "ffa"),
                                         ((130, 115, 115), (0, 1, 1), "ffa")])
def test_adjoint_passes_equal_single_iterations_3d(size, bc, obj):
    from paper_2606_31707_amd import hlbm as H
    nx, ny, nz = size
    (lx, ly, _), (hx, hy, _) = REGIONS_2D[obj](nx, ny)
    say("adjoint passes", size, bc, obj)
    a, b = (lattice(H, H.D3Q19, size, 0, bc, 0, 0.1 if obj == "ffa" else 0.0) for _ in range(2))
    for L in (a, b):
        L.set_objective(H.OBJ_FFA if obj == "ffa" else H.OBJ_DISS, (lx, ly, nz // 3), (hx, hy, nz - 1), u0=0.04)
        L.run_primal(4, accumulate=True)
    _adjoints(H, a, b, H.SOURCE_MEAN, 4, 0)
    _adjoints(H, a, b, H.SOURCE_MEAN, 2, 4)
    assert np.array_equal(a.adjoint(), b.adjoint())
    assert np.array_equal(a.gradient(), b.gradient())
    a.close()
    b.close()


def _members(H, prec, stream=None):
    """Plain, window (small region, large region, none) and adjoint members of different sizes and ends."""
    out = []
    specs = [((96, 48), (2, 1, 0), 0.0, "ffa", 0), ((61, 17), (2, 0, 0), 0.1, "diss", 1), ((130, 33), (2, 1, 0), 0.1, "ffa", 1),
             ((70, 9), (0, 1, 0), 0.0, None, 1), ((117, 40), (2, 1, 0), 0.0, "diss", 2), ((20, 30), (2, 0, 0), 0.1, "ffa", 2)]
    for i, ((nx, ny), bc, cs, obj, mode) in enumerate(specs):
        L = lattice(H, H.D2Q9, (nx, ny, 1), prec, bc, 0, cs, seed=i, **({} if stream is None else {"stream": stream}))
        if obj:
            lo, hi = REGIONS_2D[obj](nx, ny)
            L.set_objective(H.OBJ_FFA if obj == "ffa" else H.OBJ_DISS, lo, hi, u0=0.04)
        L.run_primal(2)
        if mode == 2:
            L.solve_adjoint(H.SOURCE_STEADY, turb=H.TURB_FROZEN, max_iters=0)
        out.append((L, mode))
    return out


def _same(H, a, b, where):
    for i, ((A, mode), (B, _)) in enumerate(zip(a, b)):
        assert np.array_equal(A.populations(), B.populations()), (where, i)
        if mode == 1:
            for f in (H.FIELD_MEAN_RHO, H.FIELD_MEAN_U):
                assert np.array_equal(A.field(f), B.field(f)), (where, i)
            if i != 3:
                assert A.objective(1) == B.objective(1), (where, i)
        if mode == 2:
            assert np.array_equal(A.gradient(), B.gradient()), (where, i)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("own_stream", [False, True])
def test_packed_passes_equal_packed_single_steps(prec, own_stream):
    """Runs with odd and even remainders, replayed graphs, members that a run outside the group
    left in their other array, and primal members at different parities (single steps)."""
    import torch
    from paper_2606_31707_amd import hlbm as H
    stream = torch.cuda.Stream() if own_stream else None
    h = stream.cuda_stream if own_stream else None
    say("packed passes", prec, own_stream)
    a, b = _members(H, prec, h), _members(H, prec, h)
    ga, gb = (H.Group(h) if own_stream else H.Group() for _ in range(2))
    for g, m in ((ga, a), (gb, b)):
        g.set([L for L, _ in m], [mode for _, mode in m])
    for n in (2, 7, 20, 20, 18, 3, 20, 20):
        ga.step(n)
        for _ in range(n):
            gb.step(1)
        ga.synchronize()
        gb.synchronize()
        _same(H, a, b, n)
    # a run outside the group ends in the other array; the reset brings the step count back
    for m in (a, b):
        L = m[0][0]
        u = np.zeros((3, L.n))
        L.run_primal(2)
        L.init_equilibrium(1.0, u)
    for g, m in ((ga, a), (gb, b)):
        g.set([L for L, mode in m if mode < 2], [mode for _, mode in m if mode < 2])
    for m in (a, b):
        L = m[0][0]
        L.run_primal(2)
        L.init_equilibrium(1.01, u)
    ga.step(6)
    for _ in range(6):
        gb.step(1)
    ga.synchronize()
    gb.synchronize()
    _same(H, a[:4], b[:4], "moved")
    # members at different parities
    for m in (a, b):
        m[1][0].run_primal(1)
    for g, m in ((ga, a), (gb, b)):
        g.set([L for L, mode in m if mode < 2], [mode for _, mode in m if mode < 2])
    ga.step(5)
    for _ in range(5):
        gb.step(1)
    ga.synchronize()
    gb.synchronize()
    _same(H, a[:4], b[:4], "parity")
    for m in (a, b):
        for L, _ in m:
            L.close()


@pytest.mark.parametrize("dim", [2, 3])
def test_captured_steps_replay_between_runs_with_passes(dim):
    """A captured run works on the same array at every replay, whatever runs (odd and even numbers
    of passes, a steady stop between two passes) come in between."""
    import torch
    from paper_2606_31707_amd import hlbm as H
    size = (70, 30, 1) if dim == 2 else (70, 15, 6)
    stream = torch.cuda.Stream()
    a = lattice(H, H.D2Q9 if dim == 2 else H.D3Q19, size, 1, (2, 1, 0), 0, 0.0, stream=stream.cuda_stream)
    b = lattice(H, H.D2Q9 if dim == 2 else H.D3Q19, size, 1, (2, 1, 0), 0, 0.0)
    a.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.run_primal(2)
    for steps in (0, 4, 2, 12, 6, 10, 8):
        say("captured steps", dim, steps)
        if steps:
            a.run_primal(steps)
            b.run_primal(steps)
        a.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        b.run_primal(2)
        assert np.array_equal(a.populations(), b.populations()), steps
    a.run_primal(400, steady_tol=1.0, check_every=4)  # stops after one pass
    b.run_primal(4)
    with torch.cuda.stream(stream):
        graph.replay()
    stream.synchronize()
    b.run_primal(2)
    assert np.array_equal(a.populations(), b.populations())
    a.close()
    b.close()
