"""Pair counts do not depend on the unit of length, down to separations whose
squares are near the smallest normal FP32 numbers and up to boxes whose
diagonal squared is past the largest."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2408_03036_amd import catalogs as C
from paper_2408_03036_amd import tpcf as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    T.load()
    return _t


def counts_at(torch, scale, lo, hi, spacing, nmu):
    """Counts of 700 points in a box of 1.03 scale, and the oracle's at scale 1
    (a power of two changes no rounding in double precision)."""
    box = 1.03
    pos = C.poisson(700, box, 12)
    edges = (np.geomspace if spacing == "log" else np.linspace)(lo * box, hi * box, 7)
    ref = O.xi_counts(pos, box, edges, nmu)
    h = T.Handle(box * scale, edges * scale, 0)
    h.build_grid(torch.from_numpy(pos * scale).cuda())
    got = h.xi_count(nmu).cpu().numpy()
    h.close()
    return got, ref


# one cell (every pair tested) and a stencil; nmu odd: a direction of no length
# at all falls in the middle of a bin, where no guard band sends it to FP64
@pytest.mark.parametrize("lo,hi", [(0.05, 0.45), (0.05, 0.3)])
@pytest.mark.parametrize("spacing", ["linear", "log"])
@pytest.mark.parametrize("nmu", [5, 8])
def test_squares_past_the_largest_float(torch, lo, hi, spacing, nmu):
    got, ref = counts_at(torch, 2.0**65, lo, hi, spacing, nmu)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("spacing", ["linear", "log"])
@pytest.mark.parametrize("lo,hi", [(0.05, 0.45), (0.05, 0.3)])
def test_separations_below_1e15(torch, lo, hi, spacing):
    got, ref = counts_at(torch, 2.0**-50, lo, hi, spacing, 7)
    assert np.array_equal(got, ref)
