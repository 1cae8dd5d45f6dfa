"""lbm_footprint counts what a batch slot holds: populations in whole storage
blocks, the x-band copy, velocity planes, four history buffers and the
interface tables -- of which D3Q19 keeps no ring tables, its ring kernels find
nodes and stencils from the geometry."""
import pytest

from paper_2004_11863_amd import lbm


def _expected(D, hrr, sb, n, lo, hi):
    Q = 9 if D == 2 else 19
    m = [b - a for a, b in zip(lo, hi)]
    nf = [2 * k + 1 for k in m]
    xo = 16 // sb - 1

    def padded(dims, off):
        p = (dims[0] + off + 3) // 4 * 4
        for k in dims[1:]:
            p *= k
        return p

    def prod(v):
        p = 1
        for k in v:
            p *= k
        return p

    pc, pf = padded(n, 0), padded(nf, xo)
    block = 32768 // sb
    pops = lambda p: sb * (p // block + 1) * block * Q  # noqa: E731
    total = 2 * pops(pc) + (3 if D == 2 and not hrr else 2) * pops(pf)
    if D == 3 and not hrr:
        total += sb * 2 * Q * 5 * nf[1] * nf[2]
    if hrr:
        total += sb * (1 + D) * (pc + pf + 128)
    nh = sum(2 * prod(m[b] + 3 for b in range(D) if b != a) for a in range(D))
    nt = prod(k - 1 for k in m) - prod(k - 3 for k in m)
    fields = 1 + D + Q + (3 if D == 2 else 6)
    total += 4 * 8 * fields * nh + 8 * nh + 16 * nt
    if D == 2:
        total += 76 * (prod(nf) - prod(k - 2 for k in nf))
    return total


@pytest.mark.parametrize("model", ["RR", "HRR"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,lo,hi", [((64, 50), (10, 12), (50, 40)), ((40, 30, 28), (8, 7, 6), (30, 22, 20))])
def test_footprint(model, prec, n, lo, hi):
    D = len(n)
    d = lbm.make_desc(lbm.LBM_D2Q9 if D == 2 else lbm.LBM_D3Q19, lbm.LBM_RR if model == "RR" else lbm.LBM_HRR,
                      lbm.LBM_FP32_DEV if prec == "fp32" else lbm.LBM_FP64, n, lo, hi, 0.51, 0.995)
    assert lbm.lbm_footprint(d) == _expected(D, model == "HRR", 4 if prec == "fp32" else 8, n, lo, hi)
