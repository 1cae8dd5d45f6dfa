"""Device arrays of exactly a level's size are taken, one value shorter they are
refused by every entry point that sets or reads fields.  The levels are small
enough that a missing value lies in the last page of its allocation."""
import ctypes

import numpy as np
import pytest

from paper_2004_11863_amd import inputs as I

pytestmark = pytest.mark.gpu


class Arrays:
    """Device allocations of given sizes (values), optionally starting inside a larger one."""

    def __init__(self, L):
        self.L, self.owned = L, []

    def __call__(self, values, skip=0):
        p = ctypes.c_void_p()
        assert self.L.hipMalloc(ctypes.byref(p), ctypes.c_size_t(8 * (values + skip))) == 0
        assert self.L.hipMemset(p, 0, ctypes.c_size_t(8 * (values + skip))) == 0
        self.owned.append(p)
        return p.value + 8 * skip

    def put(self, a, skip=0):
        p = self(a.size, skip)
        assert self.L.hipMemcpy(ctypes.c_void_p(p), a.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(a.nbytes), 1) == 0
        return p

    def get(self, p, shape):
        a = np.empty(shape)
        assert self.L.hipMemcpy(a.ctypes.data_as(ctypes.c_void_p), ctypes.c_void_p(p), ctypes.c_size_t(a.nbytes), 2) == 0
        return a

    def free(self):
        for p in self.owned:
            assert self.L.hipFree(p) == 0


@pytest.mark.parametrize("skip", [0, 3])
def test_short_device_arrays_are_refused(skip):
    from paper_2004_11863_amd import lbm
    n, lo, hi = (21, 18), (4, 5), (15, 12)
    wl = I.Workload(geom=I.Geometry(2, (*n, 1), (*lo, 0), (*hi, 0)), U=(0.04, -0.02, 0.01),
                    pulses=[I.Pulse(center=(10.0, 9.0), A=1e-3, R=2.5)])
    L = lbm.load()
    DEV = lbm.LBM_DEVICE
    A = Arrays(L)
    g = lbm.Grid(lbm.LBM_D2Q9, lbm.LBM_RR, lbm.LBM_FP64, n, lo, hi)
    b = lbm.Batch(lbm.LBM_D2Q9, lbm.LBM_RR, lbm.LBM_FP64, 1)
    slot = b.add(n, lo, hi)
    for lv in (0, 1):
        g.set_state(lv, *I.fields(wl, lv))
        b.set_state(slot, lv, *I.fields(wl, lv))
    for lv in (0, 1):
        rho, u = I.fields(wl, lv)
        N = g.nodes(lv)
        for size in (N, 2 * N, 9 * N):  # the value that is missing shares its page with the one before it
            assert (8 * (skip + size - 1)) % 4096 != 0
        r, v = A.put(rho, skip), A.put(u, skip)
        sr, sv, sf = A(N - 1, skip), A(2 * N - 1, skip), A(9 * N - 1, skip)
        r2, v2, f2 = A(N, skip), A(2 * N, skip), A(9 * N, skip)
        calls = {
            "set_state": (lambda a, c: L.lbm_set_state(g.h, lv, a, c, DEV), (r, v), (sr, sv)),
            "batch_set_state": (lambda a, c: L.lbm_batch_set_state(b.b, slot, lv, a, c, DEV), (r, v), (sr, sv)),
            "get_macros": (lambda a, c: L.lbm_get_macros(g.h, lv, a, c, DEV), (r2, v2), (sr, sv)),
            "batch_get_macros": (lambda a, c: L.lbm_batch_get_macros(b.b, slot, lv, a, c, DEV), (r2, v2), (sr, sv)),
            "get_populations": (lambda a: L.lbm_get_populations(g.h, lv, a, DEV), (f2,), (sf,)),
            "batch_get_populations": (lambda a: L.lbm_batch_get_populations(b.b, slot, lv, a, DEV), (f2,), (sf,)),
            "set_populations": (lambda a: L.lbm_set_populations(g.h, lv, a, DEV), (f2,), (sf,)),
        }
        for name, (call, whole, short) in calls.items():
            if name == "set_populations":  # the state as it was set, before its populations are set from f2
                for got, want in zip((r2, v2, f2), (*g.get_macros(lv), g.get_populations(lv))):
                    assert np.array_equal(A.get(got, want.shape), want), lv
            assert call(*whole) == lbm.LBM_OK, (name, lv)
            for k in range(len(whole)):
                args = [*whole[:k], short[k], *whole[k + 1:]]
                assert call(*args) == lbm.LBM_EDEVICE, (name, lv, k)
                L.hipGetLastError()  # of the refused copy
        assert np.array_equal(A.get(f2, (9, N)), g.get_populations(lv))
    g.close()
    b.close()
    A.free()
