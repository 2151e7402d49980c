"""Directions of pairs an ulp short of half a box apart."""
import math

import numpy as np
import pytest

from paper_2408_03036_amd import tpcf as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    T.load()
    return _t


# boxes whose 1 / L rounds down (3, 7, 49) and up (10), and a power of two
@pytest.mark.parametrize("L", [3.0, 7.0, 49.0, 10.0, 16.0])
@pytest.mark.parametrize("axis", [0, 2])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("lmax,weighted", [(1, False), (8, True)])
def test_directions_at_half_a_box(torch, L, axis, sign, lmax, weighted):
    """The neighbour a whole period nearer than it lies in the box is on the
    other side: its direction is that of a neighbour further on, exactly, for
    both of the pair (an ulp over half a box apart, an ulp less with the
    period)."""
    w = torch.tensor([1.0, 2.0, 1.0], dtype=torch.float64).cuda() if weighted else None

    def alm(x):
        pos = np.zeros((3, 3))
        pos[1, axis] = x
        pos[2] = 0.45 * L  # 0.78 L or more from both: in no bin
        if sign < 0:
            pos[[0, 1]] = pos[[1, 0]]
        h = T.Handle(L, np.array([0.4 * L, 0.5 * L]), lmax, precision=T.PREC_FP64)
        h.build_grid(torch.from_numpy(pos).cuda(), w, 3)
        h.alm_accumulate()
        a = h.get_alm(0, 2).cpu().numpy()
        h.close()
        return a

    near, far = alm(math.nextafter(0.5 * L, L)), alm(0.55 * L)
    assert np.abs(near).max() > 0.0
    # unit vectors along an axis, of components 1 and 0 to a rounding of 1 / r
    assert np.abs(near - far).max() <= 4 * (lmax + 1) * 2.0**-52 * np.abs(far).max()
