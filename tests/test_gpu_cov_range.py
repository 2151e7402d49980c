"""Covariance and precision at the ends of the ranges they take."""
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


def a_covariance(nd, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((2 * nd + 10, nd)) * rng.uniform(0.5, 2.0, nd)
    return np.cov(x.T).reshape(nd, nd)


# an entry in the first pivot block, the last of it, the first of the next, the
# last of a part-filled one; one block, whole blocks, an odd number with a rest
@pytest.mark.parametrize("nd,masked", [(1, [0]), (20, [3]), (64, [31, 32]), (70, [0, 45, 69])])
def test_infinite_variances(torch, nd, masked):
    """Entries of infinite variance have no weight: zero rows and columns, and
    the inverse of the rest in the others. The tolerance is the one of the
    block inverse: 32 n 2^-53 times the condition number."""
    c = a_covariance(nd, nd)
    c[masked, masked] = np.inf
    rest = [i for i in range(nd) if i not in masked]
    ref = np.zeros((nd, nd))
    if rest:
        ref[np.ix_(rest, rest)] = np.linalg.inv(c[np.ix_(rest, rest)])
    nm = 3 * nd + 20
    ref *= (nm - nd - 2.0) / (nm - 1.0)
    h = T.Handle(100.0, np.linspace(0.0, 10.0, 2), 0)
    got = h.precision(torch.from_numpy(c).cuda(), nm).cpu().numpy()
    h.close()
    assert np.all(got[masked] == 0.0) and np.all(got[:, masked] == 0.0)
    if rest:
        tol = 32.0 * nd * 2.0**-53 * np.linalg.cond(c[np.ix_(rest, rest)]) * np.abs(ref).max()
        assert np.abs(got - ref).max() <= tol


@pytest.mark.parametrize("scale", [2.0**1018, 2.0**1022, 2.0**-1018])
def test_variances_near_the_ends_of_the_range(torch, scale):
    """Uncorrelated variances of 1 to 1.75 times a power of two: 1 / x in a
    rounding or two (of a denormal: in its last bit)."""
    v = (1.0 + 0.25 * (np.arange(40) % 4)) * scale
    nm = 100
    f = (nm - 40 - 2.0) / (nm - 1.0)
    h = T.Handle(100.0, np.linspace(0.0, 10.0, 2), 0)
    got = h.precision(torch.from_numpy(np.diag(v)).cuda(), nm).cpu().numpy()
    h.close()
    ref = np.diag(f / v)
    assert np.all(np.abs(got - ref) <= 4 * 2.0**-52 * np.abs(ref) + 2 * 2.0**-1074)


# 320 chunks of 64 mocks are the last that every workgroup adds up for itself
@pytest.mark.parametrize("nm", [20480, 20481, 20544])
@pytest.mark.parametrize("nd", [1, 70])
def test_many_mocks(torch, nm, nd):
    """Against numpy; sums of nm terms in FP64, as the tolerances say."""
    x = np.random.default_rng(nm + nd).standard_normal((nm, nd)) + 3.0
    h = T.Handle(100.0, np.linspace(0.0, 10.0, 2), 0)
    mean, cov = h.covariance(torch.from_numpy(x).cuda())
    h.close()
    d = x - x.mean(0)
    ref, sd = d.T @ d / (nm - 1), np.sqrt((d * d).sum(0))
    assert np.all(np.abs(mean.cpu().numpy() - x.mean(0)) <= (nm + 4) * 2.0**-53 * np.abs(x).max(0))
    assert np.all(np.abs(cov.cpu().numpy() - ref) <= 4.0 * (nm + 4) * 2.0**-53 * np.outer(sd, sd) / (nm - 1))
