"""Fields in device memory: set and read in place, with the results of host
arrays bit for bit; device pointers that kernels cannot use in place (not
aligned for doubles) are copied, as the runtime copies them."""
import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I

pytestmark = pytest.mark.gpu


def _case(D):
    n, lo, hi = ((21, 18), (4, 5), (15, 12)) if D == 2 else ((13, 14, 12), (3, 4, 2), (9, 9, 8))
    ext = lambda v: tuple(v) + (1,) * (3 - D) if v is n else tuple(v) + (0,) * (3 - D)  # noqa: E731
    geom = I.Geometry(D, ext(n), ext(lo), ext(hi))
    c = tuple(0.5 * k for k in n)
    return n, lo, hi, I.Workload(geom=geom, U=(0.04, -0.02, 0.01), pulses=[I.Pulse(center=c, A=1e-3, R=2.5)])


@pytest.mark.parametrize("D", [2, 3])
@pytest.mark.parametrize("skew", [0, 4])
def test_fields_in_device_memory(D, skew):
    import torch
    from paper_2004_11863_amd import lbm
    n, lo, hi, wl = _case(D)
    lat = lbm.LBM_D2Q9 if D == 2 else lbm.LBM_D3Q19
    L = lbm.load()

    def device(a):
        """Address of a device copy of a, `skew` bytes past an aligned one, and its owner."""
        raw = torch.empty(a.nbytes + 8, dtype=torch.uint8, device="cuda")
        raw[skew:skew + a.nbytes] = torch.from_numpy(a.reshape(-1).view(np.uint8).copy()).cuda()
        return raw.data_ptr() + skew, raw

    def host(raw, shape):
        k = int(np.prod(shape)) * 8
        return raw[skew:skew + k].cpu().numpy().view(np.float64).reshape(shape).copy()

    g = lbm.Grid(lat, lbm.LBM_RR, lbm.LBM_FP64, n, lo, hi)
    h = lbm.Grid(lat, lbm.LBM_RR, lbm.LBM_FP64, n, lo, hi)
    b = lbm.Batch(lat, lbm.LBM_RR, lbm.LBM_FP64, 2)
    slot = b.add(n, lo, hi)
    for lv in (0, 1):
        rho, u = I.fields(wl, lv)
        h.set_state(lv, rho, u)
        (pr, kr), (pu, ku) = device(rho), device(u)
        assert L.lbm_set_state(g.h, lv, pr, pu, lbm.LBM_DEVICE) == 0
        assert L.lbm_batch_set_state(b.b, slot, lv, pr, pu, lbm.LBM_DEVICE) == 0
    for k in (g, h, b):
        k.step(3)
    torch.cuda.synchronize()
    for lv in (0, 1):
        N = h.nodes(lv)
        want = (*h.get_macros(lv), h.get_populations(lv))
        for call, pops in ((lambda r, u: L.lbm_get_macros(g.h, lv, r, u, lbm.LBM_DEVICE),
                            lambda f: L.lbm_get_populations(g.h, lv, f, lbm.LBM_DEVICE)),
                           (lambda r, u: L.lbm_batch_get_macros(b.b, slot, lv, r, u, lbm.LBM_DEVICE),
                            lambda f: L.lbm_batch_get_populations(b.b, slot, lv, f, lbm.LBM_DEVICE))):
            (pr, kr), (pu, ku), (pf, kf) = (device(np.zeros(s)) for s in ((N,), (D, N), (h.Q, N)))
            assert call(pr, pu) == 0 and pops(pf) == 0
            got = (host(kr, (N,)), host(ku, (D, N)), host(kf, (h.Q, N)))
            for k, (x, y) in enumerate(zip(got, want)):
                keep = slice(None)
                if k == 2 and lv == 0:  # covered nodes do not evolve: their populations are unspecified
                    keep = h.class_map(0) != lbm.LBM_C_COVERED
                assert np.array_equal(x[..., keep], y[..., keep]), (D, skew, lv, k)
    # populations in from device memory, the history rebuilt from them
    for lv in (0, 1):
        f = h.get_populations(lv)
        h.set_populations(lv, f)
        pf, kf = device(f)
        assert L.lbm_set_populations(g.h, lv, pf, lbm.LBM_DEVICE) == 0
    g.step(2)
    h.step(2)
    for lv in (0, 1):
        for x, y in zip(g.get_macros(lv), h.get_macros(lv)):
            assert np.array_equal(x, y), (D, skew, lv)
    for k in (g, h, b):
        k.close()
