"""lb_debug_lanes gives the decisions of the step itself.

* Uniform states on a switch of c'_1 (A within rounding of 1, 4 or 9) or of
  floor(v): the reach that a step reports is that of the floors and c'_1 dumped
  for the state, on every lattice, in FP64 and FP32; in FP64 both are the
  oracle's.
* Random states on switches, with a node here and there whose momentum is tiny
  (1e-170), so that its wavefront takes the general form of the quotients, and
  states of densities around the smallest numbers: floors and c'_1 bit-exact
  against the oracle.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# dim, lattice, delta0s
LATTICES = {"line": (1, "square", (0.4, 0.5, 0.55)), "square": (2, "square", (0.0,)),
            "square_rest": (2, "square", (0.3, 0.5)), "hex": (2, "hex", (0.0,)), "hex_rest": (2, "hex", (0.3, 0.5))}


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def problem(name, d0, nx, ny, gamma, gamma2=None):
    dim, lattice, _ = LATTICES[name]
    return oracle.Problem(dim, nx, ny, gamma=gamma, bc_x=oracle.PERIODIC, bc_y=oracle.PERIODIC, delta0=d0,
                          gamma2=gamma2, hex=lattice == "hex")


def solver(lbsd, name, d0, nx, ny, gamma, prec, gamma2=None):
    dim, lattice, _ = LATTICES[name]
    return lbsd.Solver(dim, nx, ny, gamma=gamma, d0_frac=d0, lattice=lattice, precision=prec, bc_x="periodic",
                       bc_y="periodic", gamma2=gamma2)


def reach_of(f, c1):
    return int(c1) + 2 + (int(f) if f >= 0 else -int(f) - 1)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(LATTICES))
def test_reach_is_that_of_the_lanes(lbsd, name, prec):
    dim, _, d0s = LATTICES[name]
    nx, ny = (70, 1) if dim == 1 else (40, 20)
    r = np.random.default_rng(11)
    done = 0
    while done < 90:
        d0, c = float(r.choice(d0s)), int(r.integers(1, 4))
        # dyadic rho, v and e, so that the moments are exact in FP32 too; gamma puts A at c^2 but for rounding
        rho, v, e = r.integers(5, 64) / 16.0, r.integers(-8, 9) / 8.0, r.integers(9, 200) / 16.0
        gamma = 1.0 + c * c * (1.0 - d0) / (dim * e)
        if not gamma <= 1.0 + 2.0 / dim:
            continue
        done += 1
        Y = np.zeros((dim + 2, ny, nx))
        Y[0], Y[1], Y[-1] = rho, rho * v, rho * (e + 0.5 * v * v)
        s = solver(lbsd, name, d0, nx, ny, gamma, prec)
        s.init_moments(Y, 1.0)
        fx, fy, c1 = (a[0, 0] for a in s.lanes())
        if prec == "fp64":
            assert (fx, fy, c1) == tuple(a.reshape(-1)[0] for a in oracle.lanes(problem(name, d0, nx, ny, gamma), Y))
        reach = max(reach_of(fx, c1), reach_of(fy, c1))
        s.step(1)
        if reach <= 5:
            s.sync()
        else:
            with pytest.raises(lbsd.LBError):
                s.sync()
        assert s.max_reach() == reach, (gamma, d0, rho, v, e, c1)
        s.close()


@pytest.mark.parametrize("two_gas", [False, True])
@pytest.mark.parametrize("planar", [False, True])
@pytest.mark.parametrize("name", sorted(LATTICES))
def test_both_forms_bit_exact(lbsd, name, planar, two_gas):
    dim, lattice, d0s = LATTICES[name]
    if lattice == "hex" and two_gas:
        pytest.skip("the hexagonal lattice runs one gas")
    nx, ny, gamma = (5000, 1, 1.4) if dim == 1 else (250, 33, 1.4)
    g2 = 5.0 / 3.0 if two_gas else None
    r = np.random.default_rng(5)
    for d0 in d0s:
        shp = (ny, nx)
        rho = r.uniform(0.2, 2.0, shp)
        vel = [np.where(r.random(shp) < 0.3, r.integers(-2, 3, shp), r.uniform(-1.9, 1.9, shp)) for _ in range(dim)]
        if planar and dim == 2:
            vel[1] = np.zeros(shp)
        A = np.where(r.random(shp) < 0.5, r.choice([1.0, 4.0, 9.0], shp), r.uniform(0.0, 12.0, shp))
        e = A * (1.0 - d0) / (dim * (gamma - 1.0))
        Y = np.stack([rho, *[rho * v for v in vel], rho * (e + 0.5 * sum(v * v for v in vel))])
        odd = r.random(shp) < 0.004
        Y[1] = np.where(odd, 1e-170, Y[1])
        if two_gas:
            Y = np.concatenate([Y, (rho * r.choice([0.0, 1.0, 0.5], shp))[None]])
        P = problem(name, d0, nx, ny, gamma, g2)
        s = solver(lbsd, name, d0, nx, ny, gamma, "fp64", g2)
        s.init_moments(Y, 1.0)
        for got, ref in zip(s.lanes(), oracle.lanes(P, Y)):
            assert np.array_equal(np.asarray(got).reshape(-1), np.asarray(ref).reshape(-1))
        s.close()


@pytest.mark.parametrize("name", sorted(LATTICES))
def test_tiny_densities_bit_exact(lbsd, name):
    dim, _, d0s = LATTICES[name]
    nx, ny, gamma = (4000, 1, 1.4) if dim == 1 else (250, 16, 1.4)
    r = np.random.default_rng(9)
    for d0 in d0s:
        shp = (ny, nx)
        rho = 10.0 ** r.uniform(-322.0, -300.0, shp)
        e = r.uniform(0.0, 12.0, shp) * (1.0 - d0) / (dim * (gamma - 1.0))
        Y = np.stack([rho, *[rho * r.uniform(-1.9, 1.9, shp) for _ in range(dim)], rho * (e + 1.0)])
        s = solver(lbsd, name, d0, nx, ny, gamma, "fp64")
        s.init_moments(Y, 1.0)
        for got, ref in zip(s.lanes(), oracle.lanes(problem(name, d0, nx, ny, gamma), Y)):
            assert np.array_equal(np.asarray(got).reshape(-1), np.asarray(ref).reshape(-1))
        s.close()
