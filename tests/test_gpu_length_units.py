"""Results do not depend on the unit of length: a power of two changes no
rounding anywhere, so lists, sums and multipoles have the same bits."""
import numpy as np
import pytest

from paper_2408_03036_amd import catalogs as C
from paper_2408_03036_amd import tpcf as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    T.load()
    return _t


# a box of 2e-13 units, where a stencil's volume is below the smallest FP32
# number, and one of 1e18, where it is above the largest; stencils of short
# reach and the one-cell grid
@pytest.mark.parametrize("scale", [2.0**-42, 2.0**60])
@pytest.mark.parametrize("rmax", [0.05, 0.2, 0.45])
@pytest.mark.parametrize("prec,lmax", [(T.PREC_FP64, 3), (T.PREC_FP64, 8), (T.PREC_FP32, 12),
                                       (T.PREC_MIXED_BF16X3, 4)])
def test_tiny_and_huge_units(torch, scale, rmax, prec, lmax):
    box, n = 1.03, 1500
    pos = torch.from_numpy(C.poisson(n, box, 21)).cuda()
    edges = np.linspace(0.2 * rmax * box, rmax * box, 6)
    mults = [(l, l, 0) for l in range(lmax + 1)]
    out = []
    for s in (1.0, scale):
        print(f"  scale {s} rmax {rmax} prec {prec} lmax {lmax}", flush=True)
        h = T.Handle(box * s, edges * s, lmax, precision=prec)
        h.build_grid(pos * s)
        h.alm_accumulate()
        h.contract()
        out.append((h.pair_count(), h.multipoles(mults).cpu().numpy()))
        h.close()
    assert out[0][0] == out[1][0] > 0
    assert np.array_equal(out[0][1], out[1][1])
