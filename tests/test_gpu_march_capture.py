"""A captured adjoint run reads and writes the same phi array and outlet buffers at every
replay, whatever eager adjoint runs come in between: numbers of passes with every remainder, a
stop on the criterion after an odd number of passes."""
import numpy as np
import pytest

from tests.pairs import say
from tests.test_gpu_march import lattice

pytestmark = pytest.mark.gpu


def single_iterations(H, lat, iters):
    g = H.Group()
    g.set([lat], [H.GROUP_ADJOINT])
    for _ in range(iters):
        g.step(1)
    g.synchronize()
    g.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("size,check", [((70, 30, 1), 2), ((70, 30, 1), 6), ((821, 493, 1), 4)])
def test_captured_adjoint_replays_after_an_early_stop(prec, size, check):
    """The larger lattice takes passes of four iterations."""
    import torch
    from paper_2606_31707_amd import hlbm as H
    say("captured adjoint", prec, size, check)
    nx, ny, _ = size
    stream = torch.cuda.Stream()
    a = lattice(H, H.D2Q9, size, prec, (2, 1, 0), 0, 0.0, stream=stream.cuda_stream)
    b = lattice(H, H.D2Q9, size, prec, (2, 1, 0), 0, 0.0)
    kw = dict(tau_adj=0.6, turb=H.TURB_FROZEN)
    for L in (a, b):
        # up to the outlet, whose virtual column the adjoint enters early
        L.set_objective(H.OBJ_DISS, (nx // 3, 0, 0), (nx - 2, ny - 1, 0), u0=0.04)
        L.run_primal(6, accumulate=True)
        L.solve_adjoint(H.SOURCE_MEAN, max_iters=0, **kw)
    a.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.solve_adjoint(H.SOURCE_MEAN, max_iters=2, restart=False, **kw)

    def replay():
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        single_iterations(H, b, 2)

    for iters in (0, 8, 6, 4, 12):
        if iters:
            a.solve_adjoint(H.SOURCE_MEAN, max_iters=iters, restart=False, **kw)
            single_iterations(H, b, iters)
        replay()
        assert np.array_equal(a.adjoint(), b.adjoint()), iters
    for _ in range(3):  # a criterion that holds at the first check
        it, _, st = a.solve_adjoint(H.SOURCE_MEAN, max_iters=400, tol=1e6, check_every=check, restart=False, **kw)
        assert st == H.OK and it == check
        single_iterations(H, b, check)
        assert np.array_equal(a.adjoint(), b.adjoint())
        replay()
        assert np.array_equal(a.adjoint(), b.adjoint()), "after an early stop"
        assert np.array_equal(a.gradient(), b.gradient())
    a.close()
    b.close()
