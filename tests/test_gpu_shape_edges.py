"""Kernels and dispatch branches at the sizes where they can go wrong: edges
of tiles and panels, remainders, thresholds of the rules that choose a path.
Compared with the CPU oracle, or bit for bit with another path where both must
agree."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2408_03036_amd import catalogs as C
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


# (box, outer edge, refinement, points): 64 points per cell on average is the
# last size counted cell by cell; above, cells are counted in z slabs. One-cell
# grids at 64, 65 and 1,500 points, 5^3 cells at 64 and just above.
@pytest.mark.parametrize("box,rmax,refine,n", [(100.0, 50.0, 0, 64), (100.0, 50.0, 0, 65), (100.0, 50.0, 0, 1500),
                                               (200.0, 40.0, 1, 8000), (200.0, 40.0, 1, 8001)])
@pytest.mark.parametrize("lattice", [False, True])
def test_crowded_cells_in_slabs(torch, box, rmax, refine, n, lattice):
    """The slabs keep the order by z and input index inside a cell: a crowded
    catalogue alone and in a batch whose average is far below the threshold
    (no slabs) gives the same bits, and exact counts at lmax 0. The lattice has
    many points of equal z, and points outside the box to be wrapped."""
    pos = C.dyadic_lattice(n, box, 4, 5) - box if lattice else C.poisson(n, box, 6)
    tiny = [C.poisson(3, box, 700 + i) for i in range(60)]
    sizes = [n] + [3] * len(tiny)
    edges = np.linspace(0.1 * rmax, rmax, 5)
    say(f"  slabs: n={n} box={box} refine={refine} lattice={lattice}")
    P = torch.from_numpy(pos).cuda()
    B = torch.from_numpy(np.vstack([pos] + tiny)).cuda()
    mults = O.all_multipoles(2, 2)
    h = T.Handle(box, edges, 2, precision=T.PREC_FP32, grid_refine=refine)
    one = h.run_catalogs([n], [n], P, None, mults).cpu().numpy()
    many = h.run_catalogs(sizes, sizes, B, None, mults).cpu().numpy()
    h.close()
    assert np.array_equal(one[0], many[0])
    h = T.Handle(box, edges, 0, precision=T.PREC_FP32, grid_refine=refine)
    got = h.run_catalogs([n], [n], P, None, [(0, 0, 0)]).cpu().numpy()
    h.close()
    ref, _, _ = O.run(pos, box, edges, 0, [(0, 0, 0)])
    # integer counts: only the final FP64 normalisation rounds
    assert np.abs(got[0] - ref).max() <= 1e-12 * np.abs(ref).max()


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
