"""NH sensors recorded by the fused D2Q9 kernel (k_fine2 SENS) in every tile shape:
the 64 x 8 tiles that grids take which fill the chip against the oracle, with the
bands of test_gpu_sensors, and the other shapes with the same bits."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import make_pair
from test_gpu_sensors import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,band", [("fp64", 1e-9), ("fp32", None)])
@pytest.mark.parametrize("model", ["BGK", "RR"])
def test_sensors_of_every_tile_shape(model, prec, band):
    from paper_2004_11863_amd import lbm
    p = lbm.LBM_FP64 if prec == "fp64" else lbm.LBM_FP32_DEV
    wl = I.vortex_pulse_4096(seed=3, n=512)
    g = wl.geom
    # more 32 x 8 tiles than half the CUs of the chip: variant 0 is 64 x 8
    wide = 16 // (8 if prec == "fp64" else 4)
    nf = [2 * (b - a) + 1 for a, b in zip(g.lo[:2], g.hi[:2])]
    assert -(-(-(-(nf[0] - 1) // wide)) // 30) * -(-(nf[1] - 2) // 6) >= 128
    wl.pulses = [I.Pulse(center=(g.hi[0] + 2.0, 0.5 * (g.lo[1] + g.hi[1])), A=1e-2)]
    thr, want = 1e-8, None
    for v in range(lbm.LBM_N_VARIANTS):
        gpu, ref, levels = make_pair(wl, model, p, with_oracle=v == 0)
        gpu.set_variants([0, v, 0, 0])
        lbm.lbm_sensors_enable(gpu.h, True)
        gpu.step(20)
        if v == 0:
            ref.step(20)
            for lv in levels:
                assert _compare(gpu, ref, lv, thr, band).any()
        got = [a for lv in levels for a in gpu.sensors(lv, thr)]
        gpu.close()
        want = got if want is None else want
        for a, b in zip(got, want):
            assert np.array_equal(a, b), v
