"""D3Q19 fine levels of 512 MB and more store their rows on whole 128-byte lines
(x = 0 at 31 floats or 15 doubles into a row).  The kernels that read and write
such rows against the oracle, in double at 1e-12 relative and in float at the
bars of the FP32 tests; every form of the step with the same bits."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import compare_fp32, compare_fp64, make_pair

pytestmark = pytest.mark.gpu

# patch cells: 113 x 125 x 127 fine nodes in rows of 128 doubles (116 narrow), 257 x 117 x 119 of 288 floats (260)
CELLS = {"fp64": (56, 62, 63), "fp32": (128, 58, 59)}


def _wide(nf, nbytes):
    """The level as the library stores it: 512 MB in narrow rows, and at most 12 % more in wide ones."""
    narrow = (nf[0] + 16 // nbytes - 1 + 3) // 4 * 4
    line = 128 // nbytes
    wide = (nf[0] + 2 * (line - 1)) // line * line
    return 2 * 19 * nbytes * narrow * nf[1] * nf[2] >= 512 << 20 and 100 * wide <= 112 * narrow


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("model", ["BGK", "RR", "HRR"])
def test_rows_on_whole_lines(model, prec):
    from paper_2004_11863_amd import lbm
    m = CELLS[prec]
    assert _wide([2 * k + 1 for k in m], 8 if prec == "fp64" else 4)
    lo = (3, 4, 3)
    n = tuple(k + 8 for k in m)
    hi = tuple(a + k for a, k in zip(lo, m))
    c = (hi[0] - 1.5, 0.4 * n[1], 0.6 * n[2])
    wl = I.Workload(geom=I.Geometry(3, n, lo, hi), U=(0.05, -0.02, 0.03), pulses=[I.Pulse(center=c, A=1e-3, R=3.0)],
                    vortices=[I.Vortex(center=c[:2], eps=0.01, Rc=3.0)])
    role, want = 3 if model == "HRR" else 1, None
    for v in (0, 2, 3):
        print(model, prec, "variant", v, flush=True)
        gpu, orc, levels = make_pair(wl, model, lbm.LBM_FP64 if prec == "fp64" else lbm.LBM_FP32_DEV, with_oracle=v == 0)
        var = [0, 0, 0, 0]
        var[role] = v
        gpu.set_variants(var)
        gpu.step(2)
        if v == 0:
            orc.step(2)
            if prec == "fp64":
                worst = compare_fp64(gpu, orc, levels)
                assert max(worst.values()) <= 1e-12, worst
            else:
                out = compare_fp32(gpu, orc, levels)
                assert all(e < (1e-5 if k.startswith("rho") else 1e-4) for k, e in out.items()), out
            del orc
        got = [gpu.get_populations(lv) for lv in levels]
        got[0] = got[0][:, gpu.class_map(0) != lbm.LBM_C_COVERED]
        gpu.close()
        want = got if want is None else want
        for a, b in zip(got, want):
            assert np.isfinite(a).all() and np.array_equal(a, b), v
