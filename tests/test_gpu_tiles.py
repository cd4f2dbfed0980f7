"""The step's launch shapes agree bitwise where a tile can go wrong: grids
narrower than a wave, on either side of a strip of 54 columns, and row counts
on either side of each tile height, in every storage and with every optional
feature; the oracle is the reference of one of them."""
import numpy as np
import pytest

from helpers import field_errors, fluid_mask, to_oracle
from paper_1803_01756_amd import configs, inputs, lbm

pytestmark = pytest.mark.gpu

STORAGES = [lbm.LBM_FP32_DEV, lbm.LBM_FP64, lbm.LBM_FP32_DEV_MASSEXACT]


def _fields(p, rho0, steps, seg_rows=0):
    s = lbm.Sim(p, rho0)
    if seg_rows:
        s.set_launch(seg_rows)
    s.step(steps)
    out = s.moments() + (np.array(s.health()),)
    s.close()
    return out


def _same(p, rho0, steps, shapes):
    ref = _fields(p, rho0, steps)
    for seg in shapes:
        for a, b in zip(_fields(p, rho0, steps, seg), ref):
            assert np.array_equal(a, b), (p.Nx, p.Ny, seg)
    return ref


@pytest.mark.parametrize("precision", STORAGES)
@pytest.mark.parametrize("Nx,Ny", [(3, 4), (17, 8), (53, 9), (54, 16), (55, 17), (63, 24), (64, 25),
                                   (65, 31), (109, 33), (300, 13), (1200, 130)])
def test_default_shape_equals_set_shapes(Nx, Ny, precision):
    print("\n[case] tiles %dx%d precision=%d" % (Nx, Ny, precision), flush=True)
    p = configs.channel_params(Nx, Ny, 110.0, 0.8, 2e-6, 300.0, precision, 0, g_y=-1e-5)
    rho0 = inputs.density_field(Nx, Ny, p.rho_v, 0.01, 3)
    _same(p, rho0, 7, (Ny - 2, 5, 8))


@pytest.mark.parametrize("precision", STORAGES)
@pytest.mark.parametrize("which", ["box", "gravity", "open", "cs", "props", "frozen", "single"])
def test_optional_features_over_shapes(orc, which, precision):
    print("\n[case] tiles, %s precision=%d" % (which, precision), flush=True)
    if which == "box":
        p = configs.d2_box(1.0 / 3.0, precision, N=70)
        rho0 = configs.droplet_density(p, 24.0)
    elif which == "gravity":
        p = configs.gravity_plate(75, 41, cold_band=(20, 50), precision=precision)
        rho0 = configs.initial_density(p, 4)
    elif which == "open":
        p = configs.open_channel(121, 29, p_period=90.0, precision=precision)
        rho0 = configs.initial_density(p, 5)
    elif which == "cs":
        p = configs.channel_params_cs(70, 27, 0.45, 0.8, 1e-4, 400.0, precision)
        rho0 = configs.initial_density(p, 6)
    elif which == "props":
        p = configs.channel_params(90, 35, 90.0, 0.78, 2e-5, 200.0, precision, lbm.LBM_PHASE_PROPS,
                                   lambda_l=0.6, C_v_l=3.0)
        rho0 = inputs.layer_field(90, 35, p.rho_g, p.rho_l, 12.0, 3.0, 0.01, 7)
    elif which == "frozen":
        p = configs.channel_params(90, 35, 90.0, 0.78, 2e-5, 200.0, precision, lbm.LBM_FREEZE_T)
        rho0 = configs.initial_density(p, 8)
    else:
        p = configs.channel_params(90, 35, 90.0, 0.8, 1e-5, 100.0, precision, lbm.LBM_SINGLE_PHASE,
                                   g_x=1e-5, rho_v=0.0)
        rho0 = inputs.density_field(90, 35, p.rho_g, 0.01, 9)
    got = _same(p, rho0, 40, (p.Ny, 5, 14))
    o = orc.Sim(to_oracle(orc, p), rho0)
    o.step(40)
    e = field_errors(got, o.moments(), fluid_mask(p.Nx, p.Ny, bool(p.flags & lbm.LBM_PERIODIC_Y)))
    print(e, flush=True)
    tol = (1e-10, 1e-8, 1e-10) if precision == lbm.LBM_FP64 else (1e-5, 1e-5, 1e-5)
    assert e["rho"] < tol[0] and e["u"] < tol[1] and e["T"] < tol[2]


@pytest.mark.parametrize("eos", ["rk", "cs"])
@pytest.mark.parametrize("period", [7.0, 90.5, 1e6, 0.0])
def test_inlet_density_is_the_root_of_its_pressure(eos, period):
    """The density read at the inlet column has the pressure that level n
    prescribes: P(rho, T_in) = p0 (1 + p_amp sin(2 pi n / period)), to the
    rounding of a root whose pressure is known to some 1e-15 (times the
    condition of P near the vapour spinodal, below 1e3)."""
    print("\n[case] inlet %s period=%g" % (eos, period), flush=True)
    if eos == "rk":
        p = configs.open_channel(61, 20, p_period=period, precision=lbm.LBM_FP64)
    else:
        p = configs.channel_params_cs(61, 20, precision=lbm.LBM_FP64, g_osc=0.0, period=0.0,
                                      flags=lbm.LBM_OPEN_X, p_amp=0.05, p_period=period)
    p = lbm.lbm_params_resolve(p)
    T_in = p.T_in if p.T_in > 0.0 else p.T_0
    p0 = lbm.lbm_eos_pressure(p, p.rho_v, T_in)[0]
    s = lbm.Sim(p, configs.initial_density(p, 1))
    for n in (0, 1, 2, 5, 23):
        s.step(n - s.n)
        rho = s.moments()[0][2:-2, 0]
        want = p0 * (1.0 + p.p_amp * (np.sin(2.0 * np.pi * n / period) if period > 0.0 else 1.0))
        for r in rho:
            assert abs(lbm.lbm_eos_pressure(p, r, T_in)[0] / want - 1.0) < 1e-12
    s.close()


@pytest.mark.parametrize("precision", STORAGES)
def test_heights_around_the_tallest_tiles(precision):
    print("\n[case] tall tiles precision=%d" % precision, flush=True)
    p = configs.channel_params(120, 95, 110.0, 0.8, 2e-6, 300.0, precision, 0, g_y=-1e-5)
    rho0 = inputs.density_field(120, 95, p.rho_v, 0.01, 3)
    _same(p, rho0, 6, (22, 23, 26, 27, 29, 30, 31, 93))
