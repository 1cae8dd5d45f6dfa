"""A batch replays graphs of one step and, once enough steps have been asked for,
of a run of six: calls of any length in any order, before and after the run is
captured and after the graphs are dropped, step its members as single grids."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import MODELS, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,model,prec", [(2, "RR", "fp64"), (2, "HRR", "fp32"), (3, "BGK", "fp64"), (3, "HRR", "fp32")])
def test_calls_of_any_length(D, model, prec):
    from paper_2004_11863_amd import lbm
    p = lbm.LBM_FP64 if prec == "fp64" else lbm.LBM_FP32_DEV
    n, lo, hi = ((24, 20), (5, 4), (17, 14)) if D == 2 else ((15, 14, 13), (4, 3, 3), (10, 9, 8))
    c = tuple(0.6 * k for k in n)
    wl = I.Workload(geom=I.Geometry(D, n + (1,) * (3 - D), lo + (0,) * (3 - D), hi + (0,) * (3 - D)),
                    U=(0.05, -0.02, 0.01), pulses=[I.Pulse(center=c, A=1e-3, R=2.0)])
    alone, _, levels = make_pair(wl, model, p, with_oracle=False)
    b = lbm.Batch(lbm.LBM_D2Q9 if D == 2 else lbm.LBM_D3Q19, MODELS[model][0], p, 2)
    slot = b.add(n, lo, hi)
    for lv in levels:
        b.set_state(slot, lv, *I.fields(wl, lv))
    for k, steps in enumerate((6, 7, 1, 5, 6, 25, 6, 13)):  # 24 steps asked for within the fifth call
        if k == 6:
            b.set_variants([0, 0])  # drops the graphs
        b.step(steps)
        alone.step(steps)
        for lv in levels:
            for x, y in zip(b.get_macros(slot, lv), alone.get_macros(lv)):
                assert np.isfinite(x).all() and np.array_equal(x, y), (k, steps, lv)
    assert b.slot_steps(slot) == 69
    b.close()
    alone.close()
