"""Workspace limits: what a call needs does not grow with the way its sums are
split, and results do not depend on the limit, the chunks or the grouping."""
import numpy as np
import pytest
import test_gpu_shape_edges as edges_of

from paper_2408_03036_amd import catalogs as C
from paper_2408_03036_amd import tpcf as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    assert _t.cuda.is_available(), "GPU tests need a GPU"
    T.load()
    return _t


# (catalogues, points, lmax, bins, precision, limits in MiB). The arrays of a
# call with 4,096 primaries to a partial sum fit every one of these limits; a
# buffer for the partial sums of all finer subchunks (130 MB for the first)
# does not, or not beside the catalogues' sums.
@pytest.mark.parametrize("ncat,n,lmax,nb,prec,limits", [
    (40, 2000, 10, 10, T.PREC_MIXED_BF16X3, (82, 100, 110, 150, 320)),
    (40, 2000, 4, 12, T.PREC_FP32, (42, 50, 60, 80)),
    (12, 3000, 10, 10, T.PREC_FP64, (54, 80, 120, 135))])
def test_small_workspaces(torch, ncat, n, lmax, nb, prec, limits):
    """A batch runs in each of these workspaces, and every catalogue's
    multipoles are, bit for bit, those of the step calls with room for all."""
    box, edges = 1000.0, np.linspace(24.0, 120.0, nb + 1)
    mults = [(l, l, 0) for l in range(lmax + 1)]
    pos = torch.from_numpy(np.vstack([C.poisson(n, box, 50 + c) for c in range(ncat)])).cuda()
    h = T.Handle(box, edges, lmax, precision=prec)
    alone = []
    for c in (0, ncat // 2, ncat - 1):
        h.build_grid(pos[c * n:(c + 1) * n].contiguous())
        h.alm_accumulate()
        h.contract()
        alone.append(h.multipoles(mults).cpu().numpy())
    h.close()
    for limit in limits:
        print(f"  limit {limit} MiB", flush=True)
        h = T.Handle(box, edges, lmax, precision=prec, workspace_limit=limit << 20)
        for _ in range(2):  # the second call finds the buffers of the first
            got = h.run_catalogs([n] * ncat, [n] * ncat, pos, None, mults).cpu().numpy()
            for c, ref in zip((0, ncat // 2, ncat - 1), alone):
                assert np.array_equal(got[c], ref)
        h.close()


# Partial sums held a few subchunks at a time: 14.6 MB each at 32 bins and lmax
# 16 (one at a time in the smaller workspace, all in the default one), and
# catalogues that begin and end inside such a span
@pytest.mark.parametrize("prec,isotropic,limit", [(T.PREC_FP32, False, 420), (T.PREC_FP64, True, 700)])
def test_partial_sums_in_spans(torch, prec, isotropic, limit):
    box, edges, lmax = 1000.0, np.linspace(20.0, 120.0, 33), 16
    sizes = [1500, 3, 700, 900]
    mults = [(l, l, 0) for l in range(lmax + 1)]
    flags = T.F_ISOTROPIC if isotropic else 0
    pos = torch.from_numpy(np.vstack([C.poisson(k, box, 90 + i) for i, k in enumerate(sizes)])).cuda()
    out = []
    for lim in (0, limit << 20):
        h = T.Handle(box, edges, lmax, precision=prec, flags=flags, workspace_limit=lim)
        out.append(h.run_catalogs(sizes, sizes, pos, None, mults).cpu().numpy())
        h.close()
    assert np.array_equal(out[0], out[1])


# Wide operands, whose subchunks hold 512 primaries at least: 16 bins at lmax 15
# one primary below and above the first boundary and past the second, and the
# widest operand
@pytest.mark.parametrize("n,nb,lmax", [(511, 16, 15), (513, 16, 15), (1030, 16, 15), (520, 32, 16)])
@pytest.mark.parametrize("prec,weighted", [(T.PREC_FP64, False), (T.PREC_FP32, True), (T.PREC_MIXED_BF16X6, False)])
def test_contraction_of_wide_operands(torch, n, nb, lmax, prec, weighted):
    edges_of.test_contraction_of_exported_alm(torch, n, nb, lmax, prec, weighted)


def test_no_room_at_all(torch):
    """Catalogues of one and of four subchunks in a workspace below the
    smallest lists (16 MB): refused, whatever the chunks."""
    sizes = [256, 3, 3, 900, 3]
    pos = torch.from_numpy(C.poisson(sum(sizes), 1.0, 5)).cuda()
    h = T.Handle(1.0, np.linspace(0.05, 0.5, 4), 11, workspace_limit=10 << 20)
    for _ in range(2):
        with pytest.raises(T.TpcfError) as e:
            h.run_catalogs(sizes, sizes, pos, None, [(0, 0, 0)])
        assert e.value.status == T.TPCF_ERR_ALLOC
    h.close()


def test_crowded_cells_need_no_room(torch):
    """The arrays of a grid take 96 bytes per point and 4 per work item of 16
    points; the counters of a crowded cell's slabs (0.75 bytes per point) fit
    beside them in no more room than that."""
    n = 1_000_000
    pos = torch.from_numpy(C.poisson(n, 100.0, 8)).cuda()
    h = T.Handle(100.0, np.linspace(10.0, 50.0, 3), 0, workspace_limit=int(96.5 * n))
    h.build_grid(pos)
    h.close()


@pytest.mark.parametrize("prec", [T.PREC_FP64, T.PREC_FP32, T.PREC_MIXED_BF16X6])
@pytest.mark.parametrize("nb,lmax", [(6, 4), (20, 6)])
@pytest.mark.parametrize("weighted", [False, True])
def test_isotropic_batches_equal_single_runs(torch, prec, nb, lmax, weighted):
    """Bit for bit, for catalogues that begin anywhere in the batch."""
    sizes = [257, 301, 515, 1000, 33]
    pos = [torch.from_numpy(C.poisson(n, 100.0, 60 + n)).cuda() for n in sizes]
    rng = np.random.default_rng(3)
    w = [torch.from_numpy(rng.uniform(-1.0, 1.0, n)).cuda() if weighted else None for n in sizes]
    mults = [(l, l, 0) for l in range(lmax + 1)]
    h = T.Handle(100.0, np.linspace(2.0, 40.0, nb + 1), lmax, precision=prec, flags=T.F_ISOTROPIC)
    many = h.run_catalogs(sizes, sizes, torch.cat(pos), torch.cat(w) if weighted else None, mults).cpu().numpy()
    for c, n in enumerate(sizes):
        one = h.run_catalogs([n], [n], pos[c], w[c], mults).cpu().numpy()
        assert np.array_equal(one[0], many[c])
    h.close()
