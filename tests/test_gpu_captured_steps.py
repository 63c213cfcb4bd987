"""lb_step under graph capture: a graph of an even number of steps ends in the
moment set it began with, so every replay goes on where the last one ended,
whichever number of steps a launch makes."""
import numpy as np
import pytest

from paper_1602_02675_amd import inputs

pytestmark = pytest.mark.gpu

REPLAYS = 3


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


# (dim, nx, ny, steps per graph): tubes of 8, 6 and 4 steps per launch of two nodes per lane, of 6 of five
@pytest.mark.parametrize("dim,nx,ny,n", [(1, 900, 1, 2), (1, 900, 1, 8), (1, 900, 1, 10), (1, 40000, 1, 6),
                                         (1, 100000, 1, 4), (1, 250000, 1, 6), (1, 250000, 1, 14), (2, 200, 60, 4)])
def test_replays_go_on(lbsd, dim, nx, ny, n):
    import torch

    left, right, x_d = inputs.riemann_instance(2)
    lam = inputs.cfl_lambda([left, right])
    ref = lbsd.Solver(dim, nx, ny)
    ref.init_riemann(x_d, left, right, lam=lam)
    st = torch.cuda.Stream()
    s = lbsd.Solver(dim, nx, ny, stream=st)
    s.init_riemann(x_d, left, right, lam=lam)
    s.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        s.step(n)
    for i in range(REPLAYS):
        with torch.cuda.stream(st):
            graph.replay()
        ref.step(n)
        assert np.array_equal(s.moments(), ref.moments()), i
