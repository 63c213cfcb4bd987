"""The 1-D autotuner's time per step is that of whole launches, however few
steps the admitted tubes have left."""
import pytest

from paper_1602_02675_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbsd():
    import torch

    assert torch.cuda.is_available()
    from paper_1602_02675_amd import lbsd as m

    return m


def tuned_ms(lbsd, left, n=64, nx=30000):
    p = lbsd.Pool(1, n, n * (2 * 3 * nx * 4 + 512) + (1 << 20), precision="fp32")
    for i in range(n):
        a, b, x_d = inputs.riemann_instance(i)
        assert p.admit_riemann(nx, x_d, a, b, 40 + left) is not None
    p.advance(40)
    ms = min(p.autotune(trials=9)[1] for _ in range(3))
    assert [p.poll(i) for i in (0, n - 1)] == [(40, 0), (40, 0)]
    p.close()
    return ms


@pytest.mark.parametrize("left", [1, 2])
def test_few_steps_left(lbsd, left):
    assert tuned_ms(lbsd, left) > 0.6 * tuned_ms(lbsd, 1000)
