"""The tree stage's record streams at the sizes and shapes where they can go
wrong, against the FP64 oracle on the same tree: trees at the edges of the
tiers (32, 1,024 and 16,384 vertices), a caterpillar whose open vertices exceed
the walking wave's stack (every level keeps one open), paths, hubs with more
children than a chunk of feeds, and a star with more cut vertices than the
recorded list holds (the sorting path).  Labels and cluster sizes are identical,
i_k within 1e-12, iterations within 2 and the bracket within 4 ulp (the device's
and the host's exp differ by an ulp); the all-k sweep equals the single-k calls."""
import numpy as np
import pytest

from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _random(n, seed, near=False):
    """Each vertex's parent is an earlier one (near: one of the last 40), so depths are about log n (or n / 20)."""
    rng = np.random.default_rng(seed)
    parent = np.full(n, -1, np.int32)
    lo = np.maximum(np.arange(n) - 40, 0) if near else np.zeros(n, np.int64)
    for v in range(1, n):
        parent[v] = rng.integers(lo[v], v)
    length = rng.lognormal(0.0, 0.5, n)
    length[0] = 0.0
    return parent, length


def _shuffled(parent, length, seed):
    """The same tree with its vertices renumbered (the root stays 0)."""
    n = len(parent)
    to = np.concatenate([[0], 1 + np.random.default_rng(seed).permutation(n - 1)])
    p, l = np.empty(n, np.int32), np.empty(n)
    p[to] = np.where(parent >= 0, to[np.maximum(parent, 0)], -1)
    l[to] = length
    return p, l


def _caterpillar(n, seed):
    """Spine 0, 2, 4, ..; each spine vertex has a leaf (numbered before the next spine vertex) and the next one."""
    parent = np.full(n, -1, np.int32)
    for v in range(1, n):
        parent[v] = v - 1 if v % 2 else v - 2
    length = np.random.default_rng(seed).lognormal(0.0, 0.7, n)
    length[0] = 0.0
    return parent, length


def _path(n, seed):
    length = np.random.default_rng(seed).lognormal(0.0, 0.7, n)
    length[0] = 0.0
    return np.arange(-1, n - 1, dtype=np.int32), length


def _hubs(n, hubs, seed):
    """A path of hubs, the other vertices spread over them as leaves and short branches."""
    rng = np.random.default_rng(seed)
    parent = np.full(n, -1, np.int32)
    parent[1:hubs] = np.arange(hubs - 1)
    for v in range(hubs, n):
        parent[v] = rng.integers(0, hubs) if rng.random() < 0.8 else rng.integers(hubs, v) if v > hubs else 0
    length = rng.lognormal(0.0, 0.5, n)
    length[0] = 0.0
    return _shuffled(parent, length, seed + 1)


def _star(n):
    parent = np.zeros(n, np.int32)
    parent[0] = -1
    length = np.ones(n)
    length[0] = 0.0
    return parent, length


CASES = {"random-%d" % n: (lambda n=n: _random(n, n), 3) for n in (31, 32, 33, 34, 64, 1023, 1024, 1025, 1057, 16384, 16385)}
CASES.update({
    "near-2500": (lambda: _shuffled(*_random(2500, 1, near=True), 2), 9),
    "near-40000": (lambda: _shuffled(*_random(40000, 3, near=True), 4), 12),
    "caterpillar-4001": (lambda: _caterpillar(4001, 5), 6),
    "caterpillar-200": (lambda: _caterpillar(200, 6), 4),
    "path-3000": (lambda: _path(3000, 7), 5),
    "hubs-9000": (lambda: _hubs(9000, 12, 8), 8),
    "hubs-30000": (lambda: _hubs(30000, 3, 9), 8),
    "star-6000": (lambda: _star(6000), 7),
    "star-6000-k5000": (lambda: _star(6000), 5000),
})


@pytest.mark.parametrize("name", list(CASES))
def test_tree_walk_matches_oracle(orc, name):
    import paper_1702_04739_amd as iso
    make, k = CASES[name]
    parent, length = make()
    n = len(parent)
    H.log("tree walk %s n=%d k=%d" % (name, n, k))
    ref = orc.subpartition(parent, length, k)
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k, return_clusters=True)
    assert info["sigma"] == ref.sigma and info["max_depth"] == ref.max_depth
    assert abs(ik - ref.i_k) <= 1e-12 * ref.i_k
    assert abs(info["beta"] - ref.beta) <= 4 * np.spacing(ref.beta)
    assert abs(info["iters"] - ref.iters) <= 2
    np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
    np.testing.assert_array_equal(info["cluster_size"].cpu().numpy(), ref.cl_size)
    np.testing.assert_allclose(info["cluster_den"].cpu().numpy(), ref.cl_den, rtol=1e-12, atol=0)
    if k < 100:
        ik_all, lab_all, _ = iso.subpartition_all_k(pg, lg, k)
        assert ik_all[k - 2] == ik
        np.testing.assert_array_equal(lab_all[k - 2].cpu().numpy(), ref.labels)
        _, ik2, _ = iso.isoperimetric_subpartition(pg, lg, 2)
        assert ik_all[0] == ik2


def test_tree_walk_potential(orc):
    """Full-graph style weights and a potential: predictions of the final threshold fail more often, the result does not change."""
    import paper_1702_04739_amd as iso
    parent, length = _shuffled(*_random(3000, 11, near=True), 12)
    rng = np.random.default_rng(13)
    om, p0 = rng.lognormal(0.0, 1.0, 3000), rng.lognormal(-3.0, 1.0, 3000)
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    og, qg = torch.from_numpy(om).cuda(), torch.from_numpy(p0).cuda()
    ik_all, lab_all, _ = iso.subpartition_all_k(pg, lg, 40, omega0=og, p0=qg)
    for k in (2, 3, 20, 40):
        labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k, omega0=og, p0=qg, return_clusters=True)
        assert ik == ik_all[k - 2] and torch.equal(labels, lab_all[k - 2])
        cost = (info["cluster_num"] / info["cluster_den"]).cpu().numpy()
        assert cost.max() == ik and cost.argmax() == info["jstar"]
        assert (cost <= info["beta"] * (1 + 1e-12)).all()
        assert int(info["cluster_size"].min()) >= 1


def test_tree_walk_rejects_malformed():
    """What is not a tree is refused before anything walks it: cycles beside a valid part, two roots, a self loop."""
    import paper_1702_04739_amd as iso
    parent, length = _random(5000, 14)
    for change in ({4000: 4500, 4500: 4000}, {10: -1}, {77: 77}, {3: 6000}):
        p = parent.copy()
        for v, u in change.items():
            p[v] = u
        with pytest.raises(iso._lib.IsoError):
            iso.isoperimetric_subpartition(torch.from_numpy(p).cuda(), torch.from_numpy(length).cuda(), 3)
