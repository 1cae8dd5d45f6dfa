"""The two-launch D2Q9 BGK / RR step (coarse stream + t+1/2 ring + history
capture; fused fine substeps + t+1 ring + transfer) at the edges of the
transfer's segments: a side of the TN square is cut into runs of 40 or 20
nodes by the tile shape, so patches whose sides hold one node less, exactly,
and one node more than a run are taken, square and narrow."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import compare_fp64, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mx,my", [(4, 4), (4, 43), (21, 4), (22, 23), (40, 24), (41, 42), (42, 44)])
@pytest.mark.parametrize("model", ["BGK", "RR"])
def test_transfer_segments(model, mx, my):
    from paper_2004_11863_amd import lbm
    n = (mx + 9, my + 8, 1)
    geom = I.Geometry(2, n, (3, 4, 0), (3 + mx, 4 + my, 0))
    c = (3.0 + 0.8 * mx, 4.0 + 0.3 * my)
    wl = I.Workload(geom=geom, U=(0.05, -0.02, 0.0), pulses=[I.Pulse(center=c, A=1e-3, R=2.0)],
                    vortices=[I.Vortex(center=c, eps=0.01, Rc=2.0)])
    for prec in (lbm.LBM_FP64, lbm.LBM_FP32_DEV):
        ref = None
        for v in range(lbm.LBM_N_VARIANTS):
            check = v == 0 and prec == lbm.LBM_FP64
            gpu, orc, levels = make_pair(wl, model, prec, with_oracle=check)
            gpu.set_variants([0, v, 0, 0])
            gpu.step(6)
            f = [gpu.get_populations(lv) for lv in levels]
            assert all(np.isfinite(a).all() for a in f)
            if check:
                orc.step(6)
                worst = compare_fp64(gpu, orc, levels)
                assert max(worst.values()) <= 1e-12, worst
            f[0] = f[0][:, gpu.class_map(0) != lbm.LBM_C_COVERED]
            gpu.close()
            if ref is None:
                ref = f
            for a, b in zip(f, ref):
                assert np.array_equal(a, b), (prec, v)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_tiles_by_size(prec):
    """The default takes small tiles where large ones would leave the chip idle;
    a long patch on the other side of that line equals the named tile shapes."""
    from paper_2004_11863_amd import lbm
    n, lo, hi = (1100, 60, 1), (20, 10, 0), (1063, 49, 0)
    wl = I.Workload(geom=I.Geometry(2, n, lo, hi), U=(0.05, -0.02, 0.0),
                    vortices=[I.Vortex(center=(1050.0, 40.0), eps=0.01, Rc=4.0)])
    ref = None
    for v in range(lbm.LBM_N_VARIANTS):
        gpu, _, levels = make_pair(wl, "RR", lbm.LBM_FP64 if prec == "fp64" else lbm.LBM_FP32_DEV, with_oracle=False)
        gpu.set_variants([0, v, 0, 0])
        gpu.step(4)
        f = [gpu.get_populations(lv) for lv in levels]
        f[0] = f[0][:, gpu.class_map(0) != lbm.LBM_C_COVERED]
        gpu.close()
        ref = f if ref is None else ref
        for a, b in zip(f, ref):
            assert np.isfinite(a).all() and np.array_equal(a, b), v
