"""The quick test of a row of initial densities decides as the node-by-node
check does.  Without a field the library checks rho_v node by node; a field
that holds the same value at one inner node goes through the quick test first.
Values at and around both ends of the EOS range, and around the densities
where Eq. 10 loses its real psi, for both equations of state and signs of G."""
import numpy as np
import pytest

from paper_1803_01756_amd import configs, lbm


def _refused(p, rho0):
    try:
        lbm.Sim(p, rho0).close()
    except lbm.LBMError as e:
        return e.status == lbm.LBM_EINVAL and "initial density" in str(e)
    return False


def _params(eos, G, flags):
    if eos == "cs":
        p = configs.channel_params_cs(12, 9, precision=lbm.LBM_FP64, flags=flags)
    else:
        p = configs.channel_params(12, 9, 110.0, 0.8, 0.0, 0.0, lbm.LBM_FP64, flags)
    p = lbm.lbm_params_resolve(p)
    p.G = G
    return p


def _edges(p):
    """Roots of P(rho, T_0) = rho / 3 and the ends of the EOS range."""
    rmax = (4.0 if p.flags & lbm.LBM_EOS_CS else 1.0) / p.b
    r = np.linspace(rmax * 1e-4, rmax * (1 - 1e-4), 2001)
    f = np.array([lbm.lbm_eos_pressure(p, x, p.T_0)[0] - x / 3.0 for x in r])
    out = [rmax * 1e-9, 0.999 * rmax, rmax]
    for i in np.nonzero(np.sign(f[1:]) != np.sign(f[:-1]))[0]:
        lo, hi = r[i], r[i + 1]
        for _ in range(200):
            mid = 0.5 * (lo + hi)
            fm = lbm.lbm_eos_pressure(p, mid, p.T_0)[0] - mid / 3.0
            if (fm > 0) == (f[i] > 0):
                lo = mid
            else:
                hi = mid
        out.append(0.5 * (lo + hi))
    return out


@pytest.mark.parametrize("flags", [0, lbm.LBM_PERIODIC_Y, lbm.LBM_PERIODIC_Y | lbm.LBM_FRAME_T])
@pytest.mark.parametrize("G", [-1.0, 1.0])
@pytest.mark.parametrize("eos", ["rk", "cs"])
def test_quick_test_decides_as_the_check_of_each_node(eos, G, flags):
    p = _params(eos, G, flags)
    rng = np.random.default_rng(5)
    rmax = (4.0 if eos == "cs" else 1.0) / p.b
    values = [-1.0, 5e-324, np.inf, 1e300] + list(rng.uniform(0.0, 1.05 * rmax, 40))
    for e in _edges(p):
        values += [e * (1.0 + d) for d in (0.0, 1e-15, -1e-15, 1e-13, -1e-13, 1e-10, -1e-10, 1e-6,
                                           -1e-6)]
    base = None
    seen = set()
    for v in values:
        q = lbm.lbm_params_resolve(p)
        q.rho_v, q.rho_ref = float(v), 1.0
        if not v > 0.0:
            want = True  # (rho_v <= 0 has a meaning of its own)
        else:
            # the plain nodes alone: at T_0
            q.flags &= ~(lbm.LBM_FRAME_T)
            want = _refused(q, None)
        if not want and base is None:
            base = v
        seen.add(want)
        if base is None:
            continue
        rho0 = np.full((p.Ny, p.Nx), base)
        rho0[4, 7] = v
        frame_ok = not _refused(p, np.full((p.Ny, p.Nx), base))
        assert _refused(p, rho0) == (want or not frame_ok), (eos, G, flags, v)
    rho0 = np.full((p.Ny, p.Nx), 1.0 if base is None else base)
    rho0[3, 2] = np.nan
    assert _refused(p, rho0)
    assert True in seen
