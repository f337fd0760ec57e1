"""GPU: the FP32 screen at sizes where a default call takes the distance matrix
instead (up to 4,096 points).  A flag asks for the screened rounds: without the
bounding-ball test (prune=False) they keep the neighbour lists and the final
round.  Against the FP64 oracle, on strided rows (the extra columns NaN, so that
a read past a row's coordinates shows), twice over, beside the other screens,
and the distance matrix on strided rows against the screen on the same rows;
above 4,096 points also by default, with pruned rounds and lists.
"""
import numpy as np
import pytest

from paper_1702_04739_amd import datagen
from tests import gpu_helpers as H
from tests.test_gpu_parity import CASES as SMALL

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = dict(SMALL)
CASES["uniform-n8200-d5"] = lambda: datagen.uniform(8200, 5)
CASES["c5-n4200-d128"] = lambda: datagen.config(5, n=4200)


@pytest.fixture(scope="module")
def iso():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1702_04739_amd as iso
    return iso


_cache = {}


def _oracle_tree(orc, name):
    if name not in _cache:
        X = CASES[name]()
        p, l, _, _ = orc.prim_mst(X)
        _cache[name] = (X, p, l)
    return _cache[name]


def _strided(X, extra=13):
    n, d = X.shape
    W = torch.full((n, d + extra), float("nan"), dtype=torch.float32, device="cuda")
    W[:, :d] = torch.from_numpy(X).cuda()
    return W[:, :d]


def _screened(iso, X, **kw):
    if X.shape[0] <= 4096 and "prune" not in kw and "lists" not in kw:
        kw["prune"] = False
    p, l, i = iso.mst(X, precision="fp32", **kw)
    assert i["tile_pairs"] > 0 and i["screen_precision"] == "fp32"
    return p.cpu().numpy(), l.cpu().numpy(), i


@pytest.mark.parametrize("recheck", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_fp32_screen_against_oracle(iso, orc, name, recheck):
    """FP64 recheck: the oracle's tree; FP32: up to certified near ties."""
    X, op, ol = _oracle_tree(orc, name)
    H.log("case %s n=%d d=%d fp32 screen + %s recheck" % (name, *X.shape, recheck))
    gp, gl, info = _screened(iso, torch.from_numpy(X).cuda(), recheck=recheck)
    W = ol.sum()
    if recheck == "fp64":
        np.testing.assert_array_equal(gp, op)
        np.testing.assert_allclose(gl, ol, rtol=1e-15, atol=0)
        assert abs(info["mst_weight"] - W) <= 1e-12 * max(W, 1e-300)
    else:
        if H.check_tree_vs_oracle(X, gp, op, H.screen_tol(X.shape[1])) == 0:
            np.testing.assert_array_equal(gp, op)
        assert abs(info["mst_weight"] - W) <= 1e-6 * max(W, 1e-300)


@pytest.mark.parametrize("recheck", ["fp32", "fp64"])
@pytest.mark.parametrize("kw", [{"prune": False}, {"lists": False}], ids=["lists", "no-lists"])
@pytest.mark.parametrize("name", ["c3-n1500-d784", "c1-n2000-d16", "ragged-n129-d17", "uniform-n8200-d5", "c5-n4200-d128"])
def test_fp32_screen_strided(iso, name, kw, recheck):
    X = CASES[name]()
    H.log("strided fp32 screen %s %s" % (name, kw))
    pc, lc, ic = _screened(iso, torch.from_numpy(X).cuda(), recheck=recheck, **kw)
    ps, ls, is_ = _screened(iso, _strided(X), recheck=recheck, **kw)
    np.testing.assert_array_equal(ps, pc)
    np.testing.assert_array_equal(ls, lc)
    assert ic["mst_weight"] == is_["mst_weight"]


@pytest.mark.parametrize("recheck", ["fp32", "fp64"])
@pytest.mark.parametrize("name", ["c3-n1500-d784", "c1-n2000-d16", "ragged-n129-d17"])
def test_distance_matrix_strided_equals_screen(iso, name, recheck):
    S = _strided(CASES[name]())
    p0, l0, _ = _screened(iso, S, recheck=recheck)
    p1, l1, i1 = iso.mst(S, recheck=recheck)
    assert i1["tile_pairs"] == 0
    np.testing.assert_array_equal(p1.cpu().numpy(), p0)
    np.testing.assert_array_equal(l1.cpu().numpy(), l0)


def test_fp32_screen_determinism(iso):
    X = torch.from_numpy(datagen.config(5, n=4000)).cuda()
    a, b = _screened(iso, X), _screened(iso, X)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


@pytest.mark.parametrize("cfg,n", [(1, 2000), (3, 3000), (5, 3000)])
def test_fp32_screen_among_the_screens(iso, cfg, n):
    X = torch.from_numpy(datagen.config(cfg, n=n)).cuda()
    p0, l0, _ = _screened(iso, X)
    for prec in ("bf16", "fp8") + (("int8",) if cfg == 3 else ()):
        p, l, i = iso.mst(X, precision=prec, prune=False)
        assert i["tile_pairs"] > 0
        np.testing.assert_array_equal(p.cpu().numpy(), p0)
        np.testing.assert_array_equal(l.cpu().numpy(), l0)
