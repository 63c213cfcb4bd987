"""Device memory of a pool's tables, beside its arena (no GPU needed)."""
import ctypes

import pytest


@pytest.mark.parametrize("dim,lattice,per_slot", [(1, 1, 700), (2, 2, 12000)])
def test_tables_per_slot(dim, lattice, per_slot):
    """A tile record or two per 1-D slot, 64 per 2-D one (about 170 bytes each, and the slot's own)."""
    from paper_1602_02675_amd import lbsd

    def size(slots):
        vs = lbsd.lb_velset(lattice, 0.5 if dim == 1 else 0.0)
        h = ctypes.c_void_p()
        assert lbsd._lib.lb_pool_create(dim, 1.4, ctypes.byref(vs), lbsd.LB_FP64, slots, 1 << 20, ctypes.byref(h)) == 0
        n = lbsd._lib.lb_pool_bytes(h)
        lbsd._lib.lb_pool_destroy(h)
        return n

    assert size(1 << 16) - size(1) <= per_slot * (1 << 16)
