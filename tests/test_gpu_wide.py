"""Wide, low channels, whose strips are dealt to the XCDs in chunks: widths that
leave the last chunk whole, narrow or empty (32, 33, 41 and 49 strips), with a
start that repeats nowhere, against the oracle after an odd and an even number
of steps and, in FP32, bitwise against the same channel in a pool, which deals
its tiles in runs.

Tolerances: those of the parity tests (1e-5 relative in the FP32 storages, 1e-11
on rho and T and 1e-9 on u in FP64)."""
import numpy as np
import pytest

from helpers import field_errors, fluid_mask, to_oracle
from paper_1803_01756_amd import configs, inputs, lbm

pytestmark = pytest.mark.gpu

PRECISIONS = [lbm.LBM_FP32_DEV, lbm.LBM_FP64, lbm.LBM_FP32_DEV_MASSEXACT]


def _check(orc, p, rho0, steps):
    s = lbm.Sim(p, rho0)
    o = orc.Sim(to_oracle(orc, p), rho0)
    tol = (1e-11, 1e-9, 1e-11) if p.precision == lbm.LBM_FP64 else (1e-5, 1e-5, 1e-5)
    out = []
    for n in steps:
        s.step(n)
        o.step(n)
        out.append(s.moments())
        e = field_errors(out[-1], o.moments(), fluid_mask(p.Nx, p.Ny))
        print(p.Nx, p.Ny, p.precision, s.n, e, flush=True)
        assert e["rho"] < tol[0] and e["u"] < tol[1] and e["T"] < tol[2]
    s.close()
    if p.precision == lbm.LBM_FP32_DEV:
        pool = lbm.Pool(1 << 30)
        slot = pool.admit(p, rho0, sum(steps))
        for n, ref in zip(steps, out):
            pool.run(n)
            for a, b in zip(pool.moments(slot, p.Nx, p.Ny), ref):
                assert np.array_equal(a, b)
        pool.close()


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("Nx,Ny", [(1675, 12), (1740, 40), (2210, 33), (2640, 17)])
def test_wide_channel(orc, Nx, Ny, precision):
    print("\n[case] wide %dx%d precision=%d" % (Nx, Ny, precision), flush=True)
    p = configs.channel_params(Nx, Ny, 110.0, 0.8, 2e-6, 300.0, precision, 0, g_y=-1e-5)
    _check(orc, p, inputs.density_field(Nx, Ny, p.rho_v, 0.01, Nx), (5, 6))


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("Nx,Ny", [(1740, 24), (2210, 40)])
def test_wide_open_channel(orc, Nx, Ny, precision):
    print("\n[case] wide open %dx%d precision=%d" % (Nx, Ny, precision), flush=True)
    p = configs.open_channel(Nx, Ny, p_period=300.0, precision=precision)
    _check(orc, p, inputs.density_field(Nx, Ny, p.rho_v, 0.01, Nx), (5, 6))
