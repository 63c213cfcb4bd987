"""Edges of the hexagonal step's tiles (32 x 16 nodes, a halo of 5).

Grids one node either side of a tile, a single node wide, and of more tiles
than a launch has blocks; states whose speeds c'_2 are at most 2 (one pass over
the four fields) and up to 4 (two passes of two), with and without the rest
group: against the oracle, one or two steps at the FP64 parity bar (1e-12 normwise,
momenta on one scale) and in FP32 within 2e-5 (a few FP32 roundings of the
state, as for the lattice's other FP32 fields).
"""
import pytest

import oracle
from paper_1602_02675_amd import inputs

from parity_helpers import TOL64, normwise_err

pytestmark = pytest.mark.gpu

BC = {"transmissive": oracle.TRANSMISSIVE, "periodic": oracle.PERIODIC}


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


SIZES = [(32, 16), (31, 17), (33, 15), (97, 49), (1, 40), (70, 1), (42, 26), (601, 450)]
STATES = {  # ranges of the velocity components and of e; steps
    "slow": (dict(vel=(-0.6, 0.6), e=(0.0, 4.0)), 2),
    "fast": (dict(vel=(-0.4, 0.4), e=(0.0, 17.0)), 1),
}


@pytest.mark.parametrize("bcx,bcy,d0", [("transmissive", "periodic", 0.0), ("periodic", "transmissive", 0.4)])
@pytest.mark.parametrize("kind", sorted(STATES))
@pytest.mark.parametrize("nx,ny", SIZES)
def test_tile_edges(lbsd, nx, ny, kind, bcx, bcy, d0):
    ranges, n = dict(STATES[kind][0]), STATES[kind][1]
    if d0:  # A grows by 1 / (1 - delta0)
        ranges["e"] = (0.0, ranges["e"][1] * (1.0 - d0))
    Y = inputs.random_state(nx * 100 + ny, 2, nx, ny, **ranges)
    P = oracle.Problem(2, nx, ny, hex=True, bc_x=BC[bcx], bc_y=BC[bcy], delta0=d0)
    ref, st, reach = oracle.run(P, Y, n)
    assert st == 0 and reach <= 5
    for prec, tol in (("fp64", TOL64), ("fp32", 2e-5)):
        s = lbsd.Solver(2, nx, ny, lattice="hex", precision=prec, bc_x=bcx, bc_y=bcy, d0_frac=d0)
        s.init_moments(Y, 1.0)
        s.step(n)
        got = s.moments()
        s.close()
        assert normwise_err(got, ref, 2) <= tol, prec
