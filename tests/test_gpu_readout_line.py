"""A read-out into pinned arrays gives the same bits on either side of the size
up to which its kernel writes them itself, and beside a running batch, where
they are copied."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1803_01756_amd import configs, lbm

pytestmark = pytest.mark.gpu


def _pinned(Nx, Ny):
    a = torch.full((4, Ny, Nx), float("nan"), dtype=torch.float64, pin_memory=True)
    return a, [ctypes.cast(a[q].data_ptr(), ctypes.POINTER(ctypes.c_double)) for q in range(4)]


@pytest.mark.parametrize("Nx,Ny,precision", [(1024, 128, lbm.LBM_FP32_DEV), (1025, 128, lbm.LBM_FP32_DEV),
                                             (331, 397, lbm.LBM_FP64), (700, 300, lbm.LBM_FP32_DEV_MASSEXACT)])
def test_channel(Nx, Ny, precision):
    print("\n[case] pinned read-out %dx%d precision=%d" % (Nx, Ny, precision), flush=True)
    p = configs.channel_params(Nx, Ny, 90.0, 0.8, 2e-6, 400.0, precision)
    s = lbm.Sim(p, configs.initial_density(p, 3))
    s.step(5)
    a, ptr = _pinned(Nx, Ny)
    assert lbm.lib().lbm_moments(ctypes.c_void_p(s.h), *ptr) == lbm.LBM_OK
    for x, y in zip(a.numpy(), s.moments()):
        assert np.array_equal(x, y)
    s.close()


@pytest.mark.parametrize("Nx,Ny", [(64, 20), (2048, 256), (2100, 256)])
def test_slot_beside_a_batch(Nx, Ny):
    """Read out three times: with the slot's own chunk as the last, beside a
    long chunk of the other slot, and after it."""
    print("\n[case] slot read-out %dx%d beside a batch" % (Nx, Ny), flush=True)
    p = configs.channel_params(Nx, Ny, 90.0, 0.8, 2e-6, 400.0)
    q = configs.channel_params(500, 100, 110.0, 0.8, 2e-6, 400.0)
    pool = lbm.Pool(2 << 30)
    slot = pool.admit(p, configs.initial_density(p, 3), 6)
    pool.admit(q, configs.initial_density(q, 4), 1 << 30)
    got = []
    for chunk in (6, 4000, 0):
        if chunk:
            pool.run(chunk)
        else:
            pool.wait(0)
        a, ptr = _pinned(Nx, Ny)
        assert lbm.lib().lbm_pool_moments(ctypes.c_void_p(pool.h), slot, *ptr) == lbm.LBM_OK
        got.append(a.numpy())
    ref = pool.moments(slot, Nx, Ny)
    pool.close()
    for a in got:
        for x, y in zip(a, ref):
            assert np.array_equal(x, y)
