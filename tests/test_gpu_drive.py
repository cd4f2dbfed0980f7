"""The oscillating drive and inlet at the ends of their period's range: an
infinite period holds the sine at its start (as sin(2 pi n / inf) = 0 does), and
one far below a step's length, whose phase no double resolves, still gives a
value between -1 and 1."""
import numpy as np
import pytest

from paper_1803_01756_amd import configs, lbm

pytestmark = pytest.mark.gpu


def _fields(p, steps):
    s = lbm.Sim(p, configs.initial_density(p, 5))
    s.step(steps)
    out = s.moments()
    s.close()
    return out


@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64, lbm.LBM_FP32_DEV_MASSEXACT])
@pytest.mark.parametrize("kind", ["drive", "inlet"])
def test_infinite_period(kind, precision):
    print("\n[case] infinite period, %s precision=%d" % (kind, precision), flush=True)
    if kind == "drive":
        p = configs.channel_params(70, 20, 110.0, 0.8, 1e-5, float("inf"), precision)
        q = configs.channel_params(70, 20, 110.0, 0.8, 0.0, 300.0, precision)
    else:
        p = configs.open_channel(131, 24, p_amp=0.1, p_period=float("inf"), precision=precision)
        q = configs.open_channel(131, 24, p_amp=0.0, p_period=300.0, precision=precision)
    for a, b in zip(_fields(p, 20), _fields(q, 20)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("period", [1e-9, 1e-13, 1e-16])
def test_period_below_a_step(period):
    """u after n steps differs from the undriven channel's by at most the sum of
    the drives, n g (a factor of two for the response's shape)."""
    print("\n[case] period %g" % period, flush=True)
    n, g = 40, 1e-5
    p = configs.channel_params(70, 20, 110.0, 0.8, g, period, lbm.LBM_FP64)
    q = configs.channel_params(70, 20, 110.0, 0.8, 0.0, 300.0, lbm.LBM_FP64)
    a, b = _fields(p, n), _fields(q, n)
    assert np.isfinite(a[1]).all() and np.abs(a[1] - b[1]).max() <= 2 * n * g
