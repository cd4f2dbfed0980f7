"""The read-out where its blocks of 64 columns x 8 rows can go wrong: grids on
either side of a block, with plates, periodic and open ends, against the
oracle; and the same values into pinned arrays (written by the kernel), into
pageable ones (copied), at an odd offset, and with arrays left out or shared."""
import ctypes as C

import numpy as np
import pytest
import torch

from helpers import field_errors, fluid_mask, to_oracle
from paper_1803_01756_amd import configs, inputs, lbm

pytestmark = pytest.mark.gpu


def _set_up(kind, Nx, Ny, precision):
    if kind == "open":
        p = configs.open_channel(Nx, Ny, p_period=90.0, precision=precision)
    else:
        flags = lbm.LBM_PERIODIC_Y if kind == "periodic" else 0
        p = configs.channel_params(Nx, Ny, 110.0, 0.8, 2e-6, 300.0, precision, flags)
    return p, inputs.density_field(Nx, Ny, p.rho_v, 0.01, 3)


def _pointer(a):
    return None if a is None else C.cast(a.ctypes.data, C.POINTER(C.c_double))


def _read(s, arrays):
    assert lbm.lib().lbm_moments(C.c_void_p(s.h), *[_pointer(a) for a in arrays]) == lbm.LBM_OK


@pytest.mark.parametrize("kind", ["plates", "periodic", "open"])
@pytest.mark.parametrize("Nx,Ny", [(5, 4), (63, 7), (64, 8), (65, 9), (128, 17), (130, 16)])
def test_readout_at_block_edges(orc, kind, Nx, Ny):
    print("\n[case] read-out %s %dx%d" % (kind, Nx, Ny), flush=True)
    p, rho0 = _set_up(kind, Nx, Ny, lbm.LBM_FP64)
    s = lbm.Sim(p, rho0)
    o = orc.Sim(to_oracle(orc, p), rho0)
    s.step(3)
    o.step(3)
    got = s.moments()
    e = field_errors(got, o.moments(), fluid_mask(Nx, Ny, kind == "periodic"))
    s.close()
    assert e["rho"] < 1e-10 and e["u"] < 1e-8 and e["T"] < 1e-10


@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64, lbm.LBM_FP32_DEV_MASSEXACT])
@pytest.mark.parametrize("Nx,Ny", [(5, 4), (65, 17), (200, 50)])
def test_host_memory_of_every_kind(Nx, Ny, precision):
    print("\n[case] read-out memory %dx%d precision=%d" % (Nx, Ny, precision), flush=True)
    p, rho0 = _set_up("plates", Nx, Ny, precision)
    s = lbm.Sim(p, rho0)
    s.step(5)
    n = Nx * Ny
    ref = [a.ravel() for a in s.moments()]  # pageable arrays
    # pinned, each array at an offset that is no multiple of 64 bytes
    pin = torch.full((4 * (n + 3),), -7.0, dtype=torch.float64, pin_memory=True).numpy()
    out = [pin[q * (n + 3) + 1:q * (n + 3) + 1 + n] for q in range(4)]
    _read(s, out)
    for a, b in zip(out, ref):
        assert np.array_equal(a, b)
    for q in range(4):  # nothing beside the arrays
        assert pin[q * (n + 3)] == -7.0 and (pin[q * (n + 3) + 1 + n:(q + 1) * (n + 3)] == -7.0).all()
    # one left out, one pageable; a byte offset that doubles do not have
    pin[:] = -7.0
    odd = np.zeros(8 * n + 8, np.uint8)[3:3 + 8 * n]
    _read(s, [out[0], None, odd, out[3]])
    assert np.array_equal(out[0], ref[0]) and np.array_equal(out[3], ref[3])
    assert (out[1] == -7.0).all() and np.array_equal(np.frombuffer(odd.tobytes()), ref[2])
    # one array named twice holds the later field
    _read(s, [out[0], out[1], out[1], out[0]])
    assert np.array_equal(out[0], ref[3]) and np.array_equal(out[1], ref[2])
    s.close()
