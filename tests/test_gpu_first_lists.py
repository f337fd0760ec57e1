"""GPU: neighbour lists built by the first round's screen (pruned calls).

A row's list holds every point up to its threshold, or the threshold it is
judged by is lower; rows whose list cannot decide them are screened.  So the
tree must be the one that screening every round builds, bit for bit (parent
array and FP64 lengths): at the smallest number of tiles, with a last tile of
one point, with pair bounds, with one share of the tile pairs and with several,
with more equal points than a list holds, where every distance ties, and where
the bound is too loose for lists.
"""
import numpy as np
import pytest

from paper_1702_04739_amd import datagen
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def iso():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1702_04739_amd as iso
    return iso


def _copies(n, d, sizes, seed):
    """Points of which some have `sizes` copies: lists of equal distances longer than a list."""
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d)).astype(np.float32)
    at = 0
    for m in sizes:
        X[at:at + m] = X[at]
        at += m
    return X[rng.permutation(n)]


def _clumps(n, d, m, seed):
    """Clumps of m points, far apart: a row's sampled tiles hold mostly other clumps."""
    rng = np.random.default_rng(seed)
    c = 40.0 * rng.standard_normal((-(-n // m), d))
    return (c[np.arange(n) // m] + rng.standard_normal((n, d))).astype(np.float32)


# name: (points, screen, pair bounds, whether a round has to be decided by lists)
CASES = {
    "normal-n7937-d24": (lambda: np.random.default_rng(1).standard_normal((7937, 24)).astype(np.float32), "fp32", None, True),
    "normal-n8193-d24": (lambda: np.random.default_rng(2).standard_normal((8193, 24)).astype(np.float32), "fp32", None, True),
    "uniform-n21000-d3": (lambda: datagen.uniform(21000, 3), "fp32", None, True),
    "clumps-n12000-d16": (lambda: _clumps(12000, 16, 300, 3), "fp32", None, True),
    "clumps-n9000-d40": (lambda: _clumps(9000, 40, 1000, 4), "bf16", None, False),
    "copies-n8800-d6": (lambda: _copies(8800, 6, (129, 400, 2000), 5), "fp32", None, False),
    "lattice-100x100": (lambda: datagen.lattice(100, 2), "fp32", None, False),
    "c3-n9000-d784": (lambda: datagen.config(3, n=9000), "int8", None, True),
    "c3-n9001-d784": (lambda: datagen.config(3, n=9001), "bf16", None, True),
    "c4-n8400-d4096": (lambda: datagen.config(4, n=8400), "bf16", True, True),
    "pair-bounds-normal-n8200-d24": (lambda: np.random.default_rng(6).standard_normal((8200, 24)).astype(np.float32), "bf16", True, False),
    "fp8-loose-n8500-d33": (lambda: np.random.default_rng(7).standard_normal((8500, 33)).astype(np.float32), "fp8", None, False),
}


@pytest.mark.parametrize("escalate", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_first_round_lists_tree(iso, name, escalate):
    make, precision, pair_bounds, lists = CASES[name]
    X = torch.from_numpy(make()).cuda()
    kw = dict(precision=precision, recheck="fp32", escalate=escalate)
    if pair_bounds is not None:
        kw["pair_bounds"] = pair_bounds
    p0, l0, i0 = iso.mst(X, lists=False, **kw)
    H.log("%s screened rounds %s" % (name, i0))
    p1, l1, i1 = iso.mst(X, **kw)
    H.log("%s with lists      %s" % (name, i1))
    np.testing.assert_array_equal(p1.cpu().numpy(), p0.cpu().numpy())
    np.testing.assert_array_equal(l1.cpu().numpy(), l0.cpu().numpy())
    assert i0["list_rounds"] == 0
    if lists and escalate:
        assert i1["list_rounds"] >= 1, i1
