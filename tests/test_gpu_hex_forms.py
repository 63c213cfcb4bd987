"""The hexagonal step's two forms of a node's primitives give the same bits.

A wavefront with an operand whose exponent needs scaling takes IEEE quotients
for all its nodes, the others shared reciprocals.  A uniform stream along e_1
with a transverse momentum of 1e-200 at one node (far below the rounding of
everything it meets) must give what the plain stream gives.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, NY = 96, 48


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


@pytest.mark.parametrize("d0", [0.0, 0.3])
def test_forms_agree(lbsd, d0):
    r = np.random.default_rng(7)
    s = lbsd.Solver(2, NX, NY, lattice="hex", bc_x="periodic", bc_y="periodic", d0_frac=d0)
    for _ in range(16):
        rho, v, e = r.uniform(0.3, 3.0), r.uniform(-0.9, 0.9), r.uniform(0.2, 3.0)
        Y = np.empty((4, NY, NX))
        Y[0], Y[1], Y[2], Y[3] = rho, rho * v, 0.0, rho * (e + 0.5 * v * v)
        out = []
        for tiny in (0.0, 1e-200):
            Y[2, 20, 50] = tiny
            s.init_moments(Y, 1.0)
            s.step(1)
            out.append(s.moments())
        assert np.array_equal(out[0][[0, 1, 3]], out[1][[0, 1, 3]])
        assert np.max(np.abs(out[0][2] - out[1][2])) < 1e-190
    s.close()
