"""GPU: the tree stage with the caller's vertex weights and potentials
(full-graph omega of eq. 2.2, p of eq. 2.3), one k and the sweep, against the
FP64 oracle on the same tree and points: each of the two alone and both, on
trees of one piece, with upper tiers, with hubs (a vertex's fold starts from its
weight and potential in a record or in a run of feeds) and with a deep spine.
Labels and sizes equal, i_k within 1e-12."""
import numpy as np
import pytest

from tests import gpu_helpers as H
from tests.test_gpu_tree_walk import _caterpillar, _hubs, _random, _shuffled

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "random-30": lambda: _random(30, 1),
    "random-1500": lambda: _shuffled(*_random(1500, 2), 3),
    "near-3000": lambda: _shuffled(*_random(3000, 4, near=True), 5),
    "hubs-5000": lambda: _hubs(5000, 9, 6),
    "caterpillar-1301": lambda: _caterpillar(1301, 7),
}


@pytest.mark.parametrize("omega,alpha", [("full", 0.0), ("tree", 1e-5), ("full", 3e-8), ("full", 0.002)])
@pytest.mark.parametrize("name", list(CASES))
def test_weights_and_potential_match_oracle(orc, name, omega, alpha):
    import paper_1702_04739_amd as iso
    parent, length = CASES[name]()
    n = len(parent)
    X = np.random.default_rng(n).standard_normal((n, 3)).astype(np.float32)
    sigma = 0.8
    H.log("tree weights %s omega=%s alpha=%g" % (name, omega, alpha))
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    om, p0 = iso.graph_weights(torch.from_numpy(X).cuda(), sigma, alpha=alpha, omega=omega == "full")
    kmax = 7
    ik_all, lab_all, _ = iso.subpartition_all_k(pg, lg, kmax, sigma=sigma, omega0=om, p0=p0)
    for k in (2, 3, kmax):
        ref = orc.subpartition(parent, length, k, sigma=sigma, omega=omega, alpha_pot=alpha, X=X)
        labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k, sigma=sigma, omega0=om, p0=p0,
                                                          return_clusters=True)
        np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
        np.testing.assert_array_equal(lab_all[k - 2].cpu().numpy(), ref.labels)
        np.testing.assert_array_equal(info["cluster_size"].cpu().numpy(), ref.cl_size)
        assert abs(ik - ref.i_k) <= 1e-12 * ref.i_k and ik_all[k - 2] == ik
        assert info["jstar"] == ref.jstar
