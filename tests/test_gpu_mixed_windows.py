"""1-D windows with fast cold gas at one end and slow hot gas at the other.

Each class is within the halo (floor(v) = 3 with c'_1 = 0, floor(v) = 0 with
c'_1 = 3), but floor(v) of the one with c'_1 of the other is not.  A window's
outer lanes, whose sources lay outside it, hold anything after a step (the
leftmost nodes of the fast gas no mass at all); none of it may come further in
than the halo, whatever classes the window holds.  Six steps of one launch
against the oracle: FP64 at 1e-12 normwise, FP32 within 2e-5.
"""
import numpy as np
import pytest

import oracle

from parity_helpers import TOL64, normwise_err

pytestmark = pytest.mark.gpu

STEPS = 6
# (nodes, first node of a window that holds both gases, nodes of fast gas in it, of the slowing, of the heating):
# two nodes per lane (solver, 6 steps: windows of 128 nodes, 56 apart); five per lane (pool shapes of 6 and 8
# steps: windows of 320 nodes, 260 and 240 apart)
SOLVER = (300, 20, 20, 34, 50)
POOL = {3: (800, 230, 60, 100, 100), 4: (720, 200, 60, 100, 100)}


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def state(nx, at, fast, slowing, heating):
    x = np.arange(nx) - at
    v = 3.3 - 3.0 * np.clip((x - fast) / slowing, 0.0, 1.0)
    e = 0.5 * 30.0 ** np.clip((x - fast - slowing) / heating, 0.0, 1.0)
    rho = 0.5 / e  # one pressure
    return np.stack([rho, rho * v, rho * (e + 0.5 * v * v)])[:, None]


def check(got, Y, prec):
    ref, st, reach = oracle.run(oracle.Problem(1, Y.shape[2]), Y, STEPS)
    assert st == 0 and reach == 5
    assert normwise_err(got, ref, 1) <= (TOL64 if prec == "fp64" else 2e-5)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mirror", [False, True])
def test_solver(lbsd, prec, mirror):
    Y = state(*SOLVER)
    if mirror:
        Y = np.ascontiguousarray(Y[:, :, ::-1]) * np.array([1.0, -1.0, 1.0]).reshape(3, 1, 1)
    s = lbsd.Solver(1, Y.shape[2], precision=prec)
    s.init_moments(Y, 1.0)
    s.step(STEPS)
    check(s.moments(), Y, prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", sorted(POOL))
def test_pool(lbsd, shape, prec):
    Y = state(*POOL[shape])
    p = lbsd.Pool(1, max_slots=1, precision=prec, arena_bytes=1 << 20)
    p.set_shape(shape)
    slot = p.admit_moments(Y, 1.0, STEPS)
    p.advance(STEPS)
    assert p.poll(slot) == (STEPS, 1)
    check(p.moments(slot), Y, prec)
