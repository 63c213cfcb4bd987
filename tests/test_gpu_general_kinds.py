"""The square lattice's general pass with a rest level, two gases and both.

These instances keep parts of a wavefront's state in LDS and march tiles with
far classes once or twice, for some of the fields each.  Near flows, flows whose
rows move on by more than one (|v_y| > 1), and hot ones (c'_1 beyond the near
classes), with every boundary, on grids one node either side of a tile:
* against the oracle, one step at the FP64 parity bar (1e-12 normwise, momenta on
  one scale), in FP32 within 2e-5;
* the totals are the sums of the fields (1e-12 of the sums of moduli);
* a pool slot, whose tiles are cut elsewhere, and the static step have the same bits.
"""
import numpy as np
import pytest
import torch

import oracle

from paper_1602_02675_amd import inputs
from parity_helpers import TOL64, normwise_err

pytestmark = pytest.mark.gpu

BC = {"transmissive": oracle.TRANSMISSIVE, "periodic": oracle.PERIODIC, "reflecting": oracle.REFLECTING}
KINDS = {"plain": (0.0, None), "rest": (0.4, None), "gases": (0.0, 5.0 / 3.0), "both": (0.4, 5.0 / 3.0)}
STATES = {  # ranges of v_x, v_y and of A (eq. 26)
    "near": ((-0.7, 0.7), (-0.7, 0.7), (0.0, 3.9)),
    "across": ((-0.6, 0.6), (1.05, 1.9), (0.0, 3.9)),
    "hot": ((-0.6, 0.6), (-0.6, 0.6), (4.1, 15.5)),
    "mixed": ((-1.4, 1.4), (-1.4, 1.4), (0.0, 8.5)),
}


@pytest.fixture(scope="module")
def lbsd():
    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def state(nx, ny, kind, name):
    d0, g2 = KINDS[kind]
    r = np.random.default_rng(nx * 1000 + ny)
    shp = (ny, nx)
    vx, vy, A = (r.uniform(lo, hi, shp) for lo, hi in STATES[name])
    rho = r.uniform(0.2, 2.0, shp)
    e = A * (1.0 - d0) / (2.0 * (5.0 / 3.0 - 1.0 if g2 else 0.4))  # (the mixture's A is at most this)
    Y = np.stack([rho, rho * vx, rho * vy, rho * (e + 0.5 * (vx * vx + vy * vy))])
    return np.concatenate([Y, (rho * r.uniform(0.0, 1.0, shp))[None]]) if g2 else Y


@pytest.mark.parametrize("bcs", [("transmissive", "periodic"), ("periodic", "transmissive"),
                                 ("reflecting", "reflecting")])
@pytest.mark.parametrize("name", sorted(STATES))
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("nx,ny", [(54, 16), (55, 17), (109, 33), (163, 41)])
def test_kinds(lbsd, nx, ny, kind, name, bcs):
    d0, g2 = KINDS[kind]
    Y = state(nx, ny, kind, name)
    P = oracle.Problem(2, nx, ny, bc_x=BC[bcs[0]], bc_y=BC[bcs[1]], delta0=d0, gamma2=g2)
    ref, st, reach = oracle.run(P, Y, 1)
    assert st == 0 and reach <= 5
    for prec, tol in (("fp64", TOL64), ("fp32", 2e-5)):
        s = lbsd.Solver(2, nx, ny, precision=prec, bc_x=bcs[0], bc_y=bcs[1], d0_frac=d0, gamma2=g2)
        s.init_moments(Y, 1.0)
        s.step(1)
        got, tot = s.moments(), list(s.totals()) + ([s.species_total()] if g2 else [])
        assert normwise_err(got, ref, 2) <= tol, prec
        flat = got.reshape(got.shape[0], -1)
        assert np.all(np.abs(flat.sum(axis=1) - tot) <= 1e-12 * np.abs(flat).sum(axis=1))
        pool = lbsd.Pool(2, 1, 1 << 22, precision=prec, d0_frac=d0, gamma2=g2)
        slot = pool.admit_moments(Y, 1.0, 1, bc_x=bcs[0], bc_y=bcs[1])
        pool.advance(1)
        assert np.array_equal(pool.moments(slot), got)
        pool.close()
        dt = torch.float64 if prec == "fp64" else torch.float32
        y, z = torch.from_numpy(Y).to("cuda", dt), torch.empty(Y.shape, dtype=dt, device="cuda")
        s.step_static(y, z)
        assert np.array_equal(z.double().cpu().numpy(), got)
        s.close()


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("c1", [2, 3])
def test_planar_hot_rows_stay_alike(lbsd, kind, c1):
    """x-planar flows of far classes: the rows stay bit-identical, and rho v_y 0 but for
    what the double-length sums of mirrored lanes leave: at most 12 additions, each
    off by at most 2^-105 of partial sums below 16."""
    d0, g2 = KINDS[kind]
    nx, ny = 120, 40
    x = np.arange(nx)
    A = (c1 + 0.5) ** 2 + 0.2 * np.sin(2 * np.pi * x / nx)
    rho, u = 1.0 + 0.2 * np.cos(4 * np.pi * x / nx), (0.0 if c1 == 3 else 0.3) * np.cos(2 * np.pi * x / nx)
    e = A * (1.0 - d0) / 0.8
    row = np.stack([rho, rho * u, 0 * x, rho * (e + 0.5 * u * u)] + ([rho] if g2 else []))
    s = lbsd.Solver(2, nx, ny, bc_x="periodic", bc_y="periodic", d0_frac=d0, gamma2=g2)
    s.init_moments(np.ascontiguousarray(np.repeat(row[:, None, :], ny, axis=1)), 1.0)
    assert s.lanes()[2].min() == s.lanes()[2].max() == c1
    s.step(3)
    got = s.moments()
    s.close()
    assert np.all(got == got[:, :1, :]) and np.max(np.abs(got[2])) <= 12 * 16 * 2.0 ** -105
