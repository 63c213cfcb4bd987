"""States whose packets would leave the halo by far are refused, however far.

Planar states (v_y = 0, the square lattice's lean pass) whose floor(v_x) is a
multiple of 2^29, next to one, or beyond the range of a 32-bit integer, as a
whole field and at one node, and states of huge energy (A of eq. 26 beyond
2^62): each step must end in LB_EREACH with the state untouched.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, NY = 130, 40
SPEEDS = [2.0 ** 28, 2.0 ** 29, 2.0 ** 29 + 2, -(2.0 ** 29), 2.0 ** 30, 2.0 ** 31, 3e9, -3e9]


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def refused(lbsd, Y, prec, d0, two_gas):
    if two_gas:
        Y = np.concatenate([Y, 0.5 * Y[:1]])
    s = lbsd.Solver(2, NX, NY, precision=prec, d0_frac=d0, gamma2=5.0 / 3.0 if two_gas else None)
    s.init_moments(Y, 1.0)
    s.step(1)
    with pytest.raises(lbsd.LBError) as ei:
        s.sync()
    assert ei.value.code == lbsd.LB_EREACH
    assert s.steps_done == 0 and s.max_reach() > 5
    s.close()


def field(v, e, everywhere):
    Y = np.empty((4, NY, NX))
    Y[0], Y[1], Y[2], Y[3] = 1.0, 0.0, 0.0, 1.0
    at = (slice(None), slice(None)) if everywhere else (17, 71)
    Y[1][at] = v
    Y[3][at] = 0.5 * v * v + e
    return Y


@pytest.mark.parametrize("two_gas", [False, True])
@pytest.mark.parametrize("d0", [0.0, 0.5])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("everywhere", [True, False])
@pytest.mark.parametrize("v", SPEEDS)
def test_fast_planar_states(lbsd, v, everywhere, prec, d0, two_gas):
    refused(lbsd, field(v, 0.0, everywhere), prec, d0, two_gas)


@pytest.mark.parametrize("two_gas", [False, True])
@pytest.mark.parametrize("d0", [0.0, 0.5])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("everywhere", [True, False])
@pytest.mark.parametrize("e", [1e8, 1e22, 1e37])
def test_hot_planar_states(lbsd, e, everywhere, prec, d0, two_gas):
    refused(lbsd, field(0.0, e, everywhere), prec, d0, two_gas)
