"""FP32 variant 2 of the marching D3Q19 kernels in rows of several tiles on both
sides of the lines between tiles of 128 and of 192 nodes (512 / 513, 576 / 577
fine or coarse nodes): bit for bit the two-launch / two-pass result."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import make_pair

pytestmark = pytest.mark.gpu


def _run(wl, model, variants):
    from paper_2004_11863_amd import lbm
    gpu, _, levels = make_pair(wl, model, lbm.LBM_FP32_DEV, with_oracle=False)
    gpu.set_variants(variants)
    gpu.step(3)
    f = [gpu.get_populations(lv) for lv in levels]
    f[0] = f[0][:, gpu.class_map(0) != lbm.LBM_C_COVERED]
    gpu.close()
    return f


@pytest.mark.parametrize("m", [256, 257, 288, 289])
def test_fine_rows(m):
    n, lo, hi = (m + 10, 14, 15), (5, 4, 4), (5 + m, 9, 10)
    c = (5.3 + 0.93 * m, 6.0, 7.0)
    wl = I.Workload(geom=I.Geometry(3, n, lo, hi), U=(0.05, -0.01, 0.02), pulses=[I.Pulse(center=c, A=1e-3, R=3.0)],
                    vortices=[I.Vortex(center=c, eps=0.01)])
    for model, variants in (("RR", [0, 2, 0, 0]), ("HRR", [0, 0, 0, 2])):
        for a, b in zip(_run(wl, model, variants), _run(wl, model, [0, 0, 0, 0])):
            assert np.isfinite(a).all() and np.array_equal(a, b), model


@pytest.mark.parametrize("nx", [512, 513, 576, 577])
def test_coarse_rows(nx):
    n = (nx, 12, 13)
    c = (nx - 3.7, 6.0, 7.0)
    wl = I.Workload(geom=I.Geometry(3, n, (nx - 9, 3, 4), (nx - 4, 8, 9)), U=(0.05, -0.01, 0.02),
                    pulses=[I.Pulse(center=c, A=1e-3, R=3.0)], vortices=[I.Vortex(center=c, eps=0.01)])
    for a, b in zip(_run(wl, "HRR", [0, 0, 2, 0]), _run(wl, "HRR", [0, 0, 0, 0])):
        assert np.isfinite(a).all() and np.array_equal(a, b)
