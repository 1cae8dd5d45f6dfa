"""Interface kernels at the edges of their tiles, against the oracle in double
precision (the bar of the parity tests, 1e-12 relative).

D3Q19: ring tiles hold 32 x 8 fine nodes of a face, transfer tiles 8 x 2 TN
nodes, so patches of 4 cells (one TN node inside the rim), and of one cell less,
exactly and one more than a tile along each axis are taken.
D2Q9 H-RR: the coarse step in one pass on rows that are no whole number of
vectors (gathered row ends) and on periods narrower than a tile, with the ring
and the transfer in the launches of the tiles; batch members bit for bit."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I
from parity_util import MODELS, compare_fp64, make_pair

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _workload(D, n, lo, hi):
    geom = I.Geometry(D, tuple(n) + (1,) * (3 - D), tuple(lo) + (0,) * (3 - D), tuple(hi) + (0,) * (3 - D))
    c = [a + 0.6 * (b - a) for a, b in zip(lo, hi)]
    return I.Workload(geom=geom, U=(0.05, -0.02, 0.03), pulses=[I.Pulse(center=tuple(c), A=1e-3, R=2.0)],
                      vortices=[I.Vortex(center=tuple(c[:2]), eps=0.01, Rc=2.0)])


@pytest.mark.parametrize("m", [(4, 4, 4), (4, 17, 5), (9, 4, 16), (10, 16, 4), (15, 5, 9), (16, 9, 5), (17, 8, 10)])
@pytest.mark.parametrize("model", ["BGK", "RR", "HRR"])
def test_d3q19_faces(model, m):
    from paper_2004_11863_amd import lbm
    lo = (3, 2, 4)
    wl = _workload(3, [k + 8 for k in m], lo, [a + k for a, k in zip(lo, m)])
    gpu, orc, levels = make_pair(wl, model, lbm.LBM_FP64)
    for _ in range(2):  # read between steps: the ring is completed, then stepped on
        gpu.step(2)
        orc.step(2)
        worst = compare_fp64(gpu, orc, levels)
        assert max(worst.values()) <= TOL, worst
    gpu.close()


@pytest.mark.parametrize("n", [(13, 12), (14, 33), (61, 12), (63, 35), (126, 14), (253, 13)])
def test_d2q9_hrr_ragged_rows(n):
    from paper_2004_11863_amd import lbm
    lo, hi = (3, 4), (n[0] - 4, n[1] - 4)
    wl = _workload(2, n, lo, hi)
    for prec in (lbm.LBM_FP64, lbm.LBM_FP32_DEV):
        ref = None
        for v in range(lbm.LBM_N_VARIANTS):
            check = v == 0 and prec == lbm.LBM_FP64
            gpu, orc, levels = make_pair(wl, "HRR", prec, with_oracle=check)
            gpu.set_variants([0, 0, v, v])
            gpu.step(5)
            f = [gpu.get_populations(lv) for lv in levels]
            assert all(np.isfinite(a).all() for a in f)
            if check:
                orc.step(5)
                worst = compare_fp64(gpu, orc, levels)
                assert max(worst.values()) <= TOL, worst
            live = gpu.class_map(0) != lbm.LBM_C_COVERED
            gpu.close()
            f[0] = f[0][:, live]
            if ref is None:
                ref = f
            for a, b in zip(f, ref):
                assert np.array_equal(a, b), (prec, v)
        batch = lbm.Batch(lbm.LBM_D2Q9, MODELS["HRR"][0], prec, 3)
        slots = [batch.add(n, lo, hi), batch.add((9, 7))]  # beside a uniform grid narrower than a vector row
        for lv in (0, 1):
            batch.set_state(slots[0], lv, *I.fields(wl, lv))
        uni = _workload(2, (9, 7), (0, 0), (0, 0))
        batch.set_state(slots[1], 0, *I.fields(uni, 0))
        alone, _, _ = make_pair(uni, "HRR", prec, with_oracle=False)
        alone.step(5)
        for tile in (0, 1):
            batch.set_variants([tile, tile])
            batch.step(5) if tile == 0 else None
        got = [batch.get_populations(slots[0], lv) for lv in (0, 1)]
        got[0] = got[0][:, live]
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), prec
        assert np.array_equal(batch.get_populations(slots[1], 0), alone.get_populations(0))
        alone.close()
        batch.close()


def test_d3q19_tail_limit():
    """Small fine levels in double run the ring and the transfer beside substep
    2, large ones behind it: a patch above the limit gives the bits of the
    marching kernel, alone and in a batch that it takes over the limit."""
    from paper_2004_11863_amd import lbm
    small = _workload(3, (20, 18, 16), (3, 4, 5), (15, 13, 11))
    large = _workload(3, (78, 70, 60), (4, 5, 5), (74, 65, 55))

    def alone(wl, steps, v):
        gpu, _, levels = make_pair(wl, "RR", lbm.LBM_FP64, with_oracle=False)
        gpu.set_variants([0, v, 0, 0])
        gpu.step(steps)
        f = [gpu.get_populations(lv) for lv in levels]
        live = gpu.class_map(0) != lbm.LBM_C_COVERED
        gpu.close()
        return [f[0][:, live], f[1]], live

    b = lbm.Batch(lbm.LBM_D3Q19, lbm.LBM_RR, lbm.LBM_FP64, 2)
    slots = []
    for wl in (small, large):
        g = wl.geom
        slots.append(b.add(g.n, g.lo, g.hi, tau_coarse=0.51))
        for lv in (0, 1):
            b.set_state(slots[-1], lv, *I.fields(wl, lv))
        b.step(2)
    ref, live = alone(large, 2, 2)
    for f in (alone(large, 2, 0)[0], [b.get_populations(slots[1], 0)[:, live], b.get_populations(slots[1], 1)]):
        assert all(np.isfinite(a).all() and np.array_equal(a, r) for a, r in zip(f, ref))
    ref, live = alone(small, 4, 0)
    f = [b.get_populations(slots[0], 0)[:, live], b.get_populations(slots[0], 1)]
    assert all(np.array_equal(a, r) for a, r in zip(f, ref))
    b.close()
