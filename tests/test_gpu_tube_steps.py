"""Several 1-D steps per launch: a wavefront brings a window of a tube some
steps forward by itself (two nodes per lane and 8, 6 or 4 steps up to 32K, 56K
and 200 000 nodes, in FP32 400 000; beyond that five nodes per lane and six steps, or three of
each for two gases in FP64).

Tubes one node either side of a wavefront's share and of the lines between
these forms, with every boundary, against the oracle: a step count that is no
multiple of the launch's, at the FP64 parity bar (1e-12 normwise) and in FP32
within 2e-5.  However the steps are split between calls, and whatever tile
shape a pool has, the bits are the same; a step that fails inside a launch
leaves the state of the step before it.
"""
import ctypes

import numpy as np
import pytest

import oracle

from paper_1602_02675_amd import inputs
from parity_helpers import TOL64, normwise_err

pytestmark = pytest.mark.gpu

BC = {"transmissive": oracle.TRANSMISSIVE, "periodic": oracle.PERIODIC, "reflecting": oracle.REFLECTING}
GAMMA2 = 1.67


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def state(nx, seed, two_gas=False):
    Y = inputs.random_state(seed, 1, nx, vel=(-0.9, 0.9), e=(0.0, 3.0))
    if two_gas:
        chi = np.random.default_rng(seed + 1).uniform(0.0, 1.0, (1, nx))
        Y = np.concatenate([Y, (Y[0] * chi)[None]])
    return Y


def advance(lbsd, Y, calls, prec, bc, gamma2=None):
    s = lbsd.Solver(1, Y.shape[2], precision=prec, bc_x=bc, gamma2=gamma2)
    s.init_moments(Y, 1.0)
    for n in calls:
        s.step(n)
    got = s.moments()
    s.close()
    return got


SIZES = [1, 2, 5, 31, 32, 33, 129, 32 * 1024, 32 * 1024 + 1, 56 * 1024 + 1, 200000, 200001, 200361, 400001]


@pytest.mark.parametrize("two_gas", [False, True])
@pytest.mark.parametrize("bc", sorted(BC))
@pytest.mark.parametrize("nx", SIZES)
def test_tube_edges(lbsd, nx, bc, two_gas):
    if bc == "reflecting" and nx < 5:
        pytest.skip("a walled axis needs at least 5 nodes")
    g2 = GAMMA2 if two_gas else None
    Y = state(nx, nx, two_gas)
    P = oracle.Problem(1, nx, bc_x=BC[bc], gamma2=g2)
    ref, st, reach = oracle.run(P, Y, 9)
    assert st == 0 and reach <= 5
    got = advance(lbsd, Y, (9,), "fp64", bc, g2)
    assert normwise_err(got, ref, 1) <= TOL64
    assert np.array_equal(got, advance(lbsd, Y, (1, 5, 3), "fp64", bc, g2))
    f32 = advance(lbsd, Y, (9,), "fp32", bc, g2)
    assert normwise_err(f32, ref, 1) <= 2e-5
    assert np.array_equal(f32, advance(lbsd, Y, (2, 7), "fp32", bc, g2))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("two_gas", [False, True])
def test_pool_shapes_keep_the_bits(lbsd, two_gas, prec):
    g2 = GAMMA2 if two_gas else None
    sizes, bcs = [40, 311, 1900], ["transmissive", "periodic", "reflecting"]
    ref = [advance(lbsd, state(n, n, two_gas), (11,), prec, b, g2) for n, b in zip(sizes, bcs)]
    p = lbsd.Pool(1, max_slots=4, precision=prec, gamma2=g2, arena_bytes=1 << 20)
    for shape in range(p.shapes):
        p.set_shape(shape)
        slots = [p.admit_moments(state(n, n, two_gas), 1.0, 11, bc_x=b) for n, b in zip(sizes, bcs)]
        p.advance(11)
        for slot, r in zip(slots, ref):
            assert np.array_equal(np.asarray(p.moments(slot)).reshape(r.shape), r), shape
            p.release(slot)


@pytest.mark.parametrize("nx", [400, 200400])
def test_failed_step_inside_a_launch(lbsd, nx):
    """Expansion into near-vacuum: the front's packets outrun the halo at a step
    that is in the midst of a launch's."""
    left, right = (1.0, 0.0, 0.0, 1.0), (1e-4, 0.0, 0.0, 1e-8)
    lam = 0.8 / np.sqrt(1.4)
    P = oracle.Problem(1, nx)
    Y = oracle.to_lattice(P, oracle.riemann_moments(P, inputs.node_x(nx), left, right, 0.5), lam)
    k = 0
    while k < 200:
        Yn, st, r = oracle.step(P, Y)
        k += 1
        if r > 5:
            break
        Y = Yn
    assert 1 < k < 200
    for calls in ((k + 20,), (k - 2, 9), (k - 1, 1, 8)):
        s = lbsd.Solver(1, nx)
        s.init_riemann(0.5, left, right, lam=lam)
        for n in calls:
            s.step(n)
        with pytest.raises(lbsd.LBError) as ei:
            s.sync()
        assert ei.value.code == lbsd.LB_EREACH and s.steps_done == k - 1
        out = np.empty((3, 1, nx))
        assert lbsd._lib.lb_moments(s._h, ctypes.c_void_p(out.ctypes.data), 0) == lbsd.LB_EREACH
        assert normwise_err(out, oracle.from_lattice(P, Y, lam), 1) <= TOL64
        s.close()
