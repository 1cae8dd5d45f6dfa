"""D3Q19 BGK / RR fine levels that the marching kernel cannot address (planes or
x-band copies of 2^31 bytes in its window, on thin patches): they step with the
default variants and with any variant named, in two launches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _fields(n, org, h, period):
    """Plane waves along y and z over a mean flow; x fastest."""
    y = (org[1] + h * np.arange(n[1])) * (2 * np.pi / period[1])
    z = (org[2] + h * np.arange(n[2])) * (2 * np.pi / period[2])
    rho = np.empty((n[2], n[1], n[0]))
    rho[:] = (1.0 + 1e-3 * np.cos(3 * y)[None, :] * np.cos(z)[:, None])[:, :, None]
    u = np.empty((3, n[2], n[1], n[0]))
    u[0] = (0.04 + 0.01 * np.sin(y)[None, :] + 0.0 * z[:, None])[:, :, None]
    u[1] = -0.02
    u[2] = 0.01
    return rho.reshape(-1), u.reshape(3, -1)


# x-band copy of 2.149e9 bytes; planes of 432 MB
@pytest.mark.parametrize("cells,variants", [((4, 594, 594), ([0, 0, 0, 0], [0, 2, 0, 0], [0, 3, 0, 0])),
                                            ((600, 1180, 4), ([0, 0, 0, 0],))])
def test_levels_past_the_marching_limits(cells, variants):
    from paper_2004_11863_amd import lbm
    lo = (3, 4, 3)
    n = tuple(m + 8 for m in cells)
    hi = tuple(a + m for a, m in zip(lo, cells))
    nf = tuple(2 * m + 1 for m in cells)
    init = (_fields(n, (0, 0, 0), 1.0, n), _fields(nf, lo, 0.5, n))
    want = None
    for v in (None, *variants):
        print("patch of", cells, "cells, variants", v, flush=True)
        g = lbm.Grid(lbm.LBM_D3Q19, lbm.LBM_RR, lbm.LBM_FP64, n, lo, hi)
        for lv in (0, 1):
            g.set_state(lv, *init[lv])
        if v is not None:
            g.set_variants(v)
        g.step(2)
        got = [a for lv in (0, 1) for a in g.get_macros(lv)]
        g.close()
        if want is None:
            want = got
            assert all(np.isfinite(a).all() for a in got)
            assert np.abs(got[2] - 1.0).max() < 2e-3 and not np.array_equal(got[2], init[1][0])
        for a, b in zip(got, want):
            assert np.array_equal(a, b), v
