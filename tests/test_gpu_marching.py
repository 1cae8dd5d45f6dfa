"""The marching D3Q19 kernels (one node per lane, tiles of columns along z) at
the edges of their tiles: tiles hold 128 or 64 nodes along x in FP32, 32 or 64
in FP64, and 5 or 13 along y, and a run of planes along z.  Every variant
does the arithmetic of the two-launch / two-pass path node by node, so its
result is bitwise the same."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import make_pair

pytestmark = pytest.mark.gpu


def _workload(n, lo, hi):
    geom = I.Geometry(3, n, lo, hi)
    c = tuple(0.5 * v + 0.3 for v in n)
    return I.Workload(geom=geom, U=(0.05, -0.01, 0.02), pulses=[I.Pulse(center=c, A=1e-3, R=3.0)],
                      vortices=[I.Vortex(center=c, eps=0.01)])


def _run(wl, model, prec, variants, steps=3):
    gpu, _, levels = make_pair(wl, model, prec, with_oracle=False)
    gpu.set_variants(variants)
    gpu.step(steps)
    f = [gpu.get_populations(lv) for lv in levels]
    for k, a in enumerate(f):
        assert np.isfinite(a).all(), (model, variants, k)
    if len(levels) > 1:
        live = gpu.class_map(0) != 3  # covered coarse nodes are not evolved
        f[0] = f[0][:, live]
    gpu.close()
    return f


def _same(a, b, what):
    for k, (x, y) in enumerate(zip(a, b)):
        assert np.array_equal(x, y), (what, k)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("m", [4, 32, 33, 64, 65])
def test_fine_tile_edges(m, prec):
    from paper_2004_11863_amd import lbm
    p = lbm.LBM_FP32_DEV if prec == "fp32" else lbm.LBM_FP64
    wl = _workload((m + 12, 17, 18), (4, 4, 3), (4 + m, 12, 12))
    for model, role in (("RR", 1), ("HRR", 3)):
        var = [0, 0, 0, 0]
        ref = _run(wl, model, p, var)
        for v in (2, 3):
            var[role] = v
            _same(_run(wl, model, p, var), ref, (model, v))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx", [12, 33, 64, 65, 128, 129])
def test_coarse_one_pass_tile_edges(nx, prec):
    """The coarse H-RR step in one marching pass (periodic in every axis, TN
    nodes from the velocity planes, covered nodes skipped) against the velocity
    pass and collision, with a patch and on a uniform grid."""
    from paper_2004_11863_amd import lbm
    p = lbm.LBM_FP32_DEV if prec == "fp32" else lbm.LBM_FP64
    for lo, hi in (((3, 5, 2), (nx - 4, 14, 15)), ((0, 0, 0), (0, 0, 0))):
        wl = _workload((nx, 19, 18), lo, hi)
        ref = _run(wl, "HRR", p, [0, 0, 0, 0], steps=4)
        for v in (2, 3):
            _same(_run(wl, "HRR", p, [0, 0, v, 0], steps=4), ref, (lo, v))


@pytest.mark.parametrize("m", [64, 65, 96, 97])
def test_wide_tile_choice(m):
    """FP32 variant 2 takes tiles of 192 nodes along x in rows of 129 to 192
    nodes, of 128 on either side, fine and coarse."""
    from paper_2004_11863_amd import lbm
    wl = _workload((2 * m + 1, 17, 18), (20, 4, 3), (20 + m, 12, 12))
    ref = _run(wl, "RR", lbm.LBM_FP32_DEV, [0, 0, 0, 0])
    _same(_run(wl, "RR", lbm.LBM_FP32_DEV, [0, 2, 0, 0]), ref, "RR")
    ref = _run(wl, "HRR", lbm.LBM_FP32_DEV, [0, 0, 0, 0])
    _same(_run(wl, "HRR", lbm.LBM_FP32_DEV, [0, 0, 2, 2]), ref, "HRR")
