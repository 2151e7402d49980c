"""Kernels and dispatch branches at the sizes where they can go wrong: edges
of tiles and panels, remainders, thresholds of the rules that choose a path.
Compared with the CPU oracle, or bit for bit with another path where both must
agree."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2408_03036_amd import tpcf as T

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    T.load()
    return _t


# n = sum k^2 unknowns: 1, 5 and 30 (one panel of 32 columns, part filled), 55,
# 91, 204 and 285 (whole panels and remainders 23, 27, 12 and 29)
@pytest.mark.parametrize("lmax,nb", [(0, 2), (1, 3), (3, 3), (4, 9), (5, 2), (7, 1), (8, 1)])
def test_edge_correction_pivoting(torch, lmax, nb):
    """Random triplet counts without a dominant coefficient, so that the
    elimination exchanges rows in every panel; the tolerance is ten times the
    change of the oracle's solution when R changes by 1e-13."""
    rng = np.random.default_rng(lmax)
    box, edges, nD, nR = 100.0, np.linspace(2.0, 20.0, nb + 1), 5000, 50000
    s1 = lmax + 1

    def coefficients(scale, mono):
        X = np.zeros((s1, s1, s1, nb, nb))
        for m in range(s1):
            X[m, m:, m:] = rng.uniform(-scale, scale, (s1 - m, s1 - m, nb, nb))
        X[0, 0, 0] += mono
        return X

    N, R = coefficients(0.5, 0.0), coefficients(1.0, 0.1)
    say(f"  oracle: lmax={lmax} nb={nb}")
    ref = O.edge_correct_anisotropic(N.astype(complex), R.astype(complex)).real
    moved = O.edge_correct_anisotropic(N.astype(complex),
                                       (R * (1.0 + 1e-13 * rng.standard_normal(R.shape))).astype(complex)).real
    axes = (0, 1, 2)  # every (b1, b2) is a system of its own
    tol = 10.0 * np.abs(moved - ref).max(axes) + 1e-12 * np.abs(ref).max(axes)
    h = T.Handle(box, edges, lmax, precision=T.PREC_FP64)
    NN = torch.from_numpy(N * O.rrr(nD, box, edges)[None, None, None]).cuda()
    RR = torch.from_numpy(R * O.rrr(nR, box, edges)[None, None, None]).cuda()
    _, zeta = h.edge_correct(NN, nD, RR, nR, None, want_zeta=True)
    got = zeta.cpu().numpy()
    h.close()
    off = np.abs(got - ref).max(axes)
    say(f"  largest error over tolerance {float((off / tol).max()):.2e}")
    assert np.all(off <= tol)
