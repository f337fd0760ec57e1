"""GPU: the tree of few points from the matrix of all their exact distances.

Default FP32 calls of up to 4,096 points take it; any flag asks for the
screened rounds, so the same points give both.  Edges are totally ordered in
both, so parents, FP64 lengths and the weight have to be equal bit for bit: at
the edges of the tiles, waves and workgroups, at one coordinate, at 64 and 65
(one partial sum per lane, then more), with many equal distances, for a path and
a star (the deepest and the widest tour), strided rows, and at the largest size
and the one after it.  Points that the screened rounds refuse are refused alike.
"""
import numpy as np
import pytest

from paper_1702_04739_amd import datagen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def iso():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1702_04739_amd as iso
    return iso


def _normal(n, d, seed=0):
    return np.random.default_rng(seed + 1000 * n + d).standard_normal((n, d)).astype(np.float32)


CASES = {"normal-n%d-d%d" % (n, d): (lambda n=n, d=d: _normal(n, d))
         for n, d in ((2, 1), (3, 7), (17, 2), (63, 64), (64, 65), (65, 5), (150, 5), (129, 1000), (512, 63),
                      (777, 128), (1023, 3), (1024, 31), (1025, 33), (1500, 784), (2047, 16), (2048, 8), (2049, 70), (4095, 3), (4096, 9), (4097, 9))}
CASES.update({
    "same-n300": lambda: np.full((300, 7), 0.25, np.float32),
    "copies-n2000": lambda: np.repeat(_normal(20, 4), 100, axis=0)[np.random.default_rng(1).permutation(2000)],
    "lattice-45x45": lambda: datagen.lattice(45, 2),
    "path-n4096": lambda: np.random.default_rng(2).permutation(4096).astype(np.float32)[:, None] * np.float32(0.5),
    "star-m4000": lambda: datagen.star_points(4000, 6),
    "offset-n200-d40": lambda: _normal(200, 40) + np.float32(4096.0),
    "tiny-n100-d3": lambda: _normal(100, 3) * np.float32(1e-20),
})


@pytest.mark.parametrize("recheck", ["fp32", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_dense_tree_equals_screened(iso, name, recheck):
    X = torch.from_numpy(np.ascontiguousarray(CASES[name]())).cuda()
    p0, l0, i0 = iso.mst(X, recheck=recheck, lists=False)
    p1, l1, i1 = iso.mst(X, recheck=recheck)
    np.testing.assert_array_equal(p1.cpu().numpy(), p0.cpu().numpy())
    np.testing.assert_array_equal(l1.cpu().numpy(), l0.cpu().numpy())
    assert i1["mst_weight"] == i0["mst_weight"] and i1["screen_precision"] == "fp32"
    n = X.shape[0]
    if n <= 4096:
        assert i1["candidates"] == n * (n - 1) // 2 and i1["tile_pairs"] == 0


@pytest.mark.parametrize("d", [5, 64, 100])
def test_dense_strided_rows(iso, d):
    wide = torch.from_numpy(_normal(333, d + 3)).cuda()
    X = wide[:, 1:1 + d]
    p0, l0, _ = iso.mst(X.contiguous())
    p1, l1, _ = iso.mst(X)
    np.testing.assert_array_equal(p1.cpu().numpy(), p0.cpu().numpy())
    np.testing.assert_array_equal(l1.cpu().numpy(), l0.cpu().numpy())


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1e19, 3e38])
def test_dense_refuses_what_the_screen_refuses(iso, value):
    """A coordinate that is no number, or so large that squares overflow: the
    same error, or the same tree, as the screened rounds."""
    from paper_1702_04739_amd._lib import IsoError
    X = _normal(200, 6)
    X[77, 3] = value
    got = []
    for lists in (False, True):
        try:
            p, l, _ = iso.mst(torch.from_numpy(X).cuda(), lists=lists)
            got.append((p.cpu().numpy(), l.cpu().numpy()))
        except IsoError as e:
            got.append(e.code)
    if isinstance(got[0], tuple):
        np.testing.assert_array_equal(got[1][0], got[0][0])
        np.testing.assert_array_equal(got[1][1], got[0][1])
    else:
        assert got[1] == got[0]
