"""GPU: neighbour lists on points whose norms have heavy tails (pair bounds) and
on points with many copies, where lists are of little use: the tree is the one
that screening every round builds, bit for bit, by the same screen, and the
list rounds leave no more rows to the exact rescan than screened rounds do.
"""
import numpy as np
import pytest

from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def iso():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1702_04739_amd as iso
    return iso


def _tails(n, d, frac, mu, sigma, seed):
    """Normal points, a fraction of them at lognormal radii."""
    rng = np.random.default_rng(seed)
    r = np.where(rng.random((n, 1)) < frac, rng.lognormal(mu, sigma, (n, 1)), 1.0)
    return (rng.standard_normal((n, d)) * r).astype(np.float32)


def _same_tree(iso, X, lists, **kw):
    """lists: whether a round has to be decided by lists (None: either)."""
    X = torch.from_numpy(np.ascontiguousarray(X)).cuda()
    p0, l0, i0 = iso.mst(X, lists=False, **kw)
    H.log("screened   %s" % i0)
    p1, l1, i1 = iso.mst(X, **kw)
    H.log("with lists %s" % i1)
    np.testing.assert_array_equal(p1.cpu().numpy(), p0.cpu().numpy())
    np.testing.assert_array_equal(l1.cpu().numpy(), l0.cpu().numpy())
    assert i1["screen_precision"] == i0["screen_precision"] and i1["pair_bounds"] == i0["pair_bounds"]
    assert i1["rescanned_rows"] <= i0["rescanned_rows"]
    if lists is not None:
        assert (i1["list_rounds"] > 0) == lists, i1


@pytest.mark.parametrize("recheck", ["fp32", "fp64"])
@pytest.mark.parametrize("n,frac,mu,sigma", [(30000, 0.3, 1.0, 0.5), (50000, 0.02, 2.0, 1.0)])
def test_rows_without_a_listed_bound(iso, n, frac, mu, sigma, recheck):
    """A component far out whose rows list only each other: every row is undecided and has no bound yet."""
    _same_tree(iso, _tails(n, 64, frac, mu, sigma, n), True, precision="bf16", recheck=recheck)


@pytest.mark.parametrize("n,sigma", [(8200, 0.25), (20000, 0.5), (50000, 1.0)])
def test_no_lists_where_the_first_round_joins_nearly_all(iso, n, sigma):
    """Every point's nearest point lies further inwards: next to no pairs of mutually nearest points."""
    _same_tree(iso, _tails(n, 64, 1.0, 0.0, sigma, n), False, precision="bf16", pair_bounds=True)


def _half_copies(n, d, spread, seed):
    """Half of the points at one place: copies, or as near as `spread`."""
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d))
    X[: n // 2] = 0.37 + spread * X[: n // 2]
    return X[rng.permutation(n)].astype(np.float32)


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("n,d,spread", [(8200, 16, 0.0), (9001, 33, 1e-6), (12000, 8, 1e-3)])
def test_rows_that_flood_their_list(iso, n, d, spread, precision):
    """More (nearly) equal distances in a tile than a list is offered before it is cut to below its dropped values."""
    _same_tree(iso, _half_copies(n, d, spread, n), None, precision=precision)


@pytest.mark.parametrize("n,d,scale", [(8300, 6, 2e18), (9000, 24, 1.6e18), (9000, 24, 1e18)])
def test_listed_upper_bounds_of_large_distances(iso, n, d, scale):
    """Squared distances within their error bound of the largest float: a listed pair's upper bound stays one."""
    X = np.random.default_rng(1000 * n + d).standard_normal((n, d)).astype(np.float32) * np.float32(scale)
    _same_tree(iso, X, True, precision="bf16", recheck="fp64", pair_bounds=True)
