"""GPU: more cut vertices than the recorded list holds (4,096), the path that
sorts the vertices, where the other tests do not reach it: several such k of
one all-k sweep beside one that is not, and costs below -1.  Against the FP64
oracle: labels equal, i_k within 1e-12.
"""
import numpy as np
import pytest

from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _two_stars(a, b):
    """Hub 0 with a leaves and hub 1, which has b leaves; every edge of length 1."""
    parent = np.concatenate([[-1, 0], np.zeros(a), np.ones(b)]).astype(np.int32)
    length = np.ones(len(parent))
    length[0] = 0.0
    return parent, length


def test_sorted_cuts_in_a_sweep(orc):
    import paper_1702_04739_amd as iso
    parent, length = _two_stars(2500, 4000)
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    H.log("sorted cuts in a sweep n=%d" % len(parent))
    ik_all, lab_all, _ = iso.subpartition_all_k(pg, lg, 6)
    for k in range(2, 7):
        ref = orc.subpartition(parent, length, k)
        labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k)
        np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
        np.testing.assert_array_equal(lab_all[k - 2].cpu().numpy(), ref.labels)
        assert abs(ik - ref.i_k) <= 1e-12 * ref.i_k and ik_all[k - 2] == ik and info["jstar"] == ref.jstar


def test_sorted_cuts_costs_below_minus_one(orc):
    """Flows of one; 4,200 leaves of potential -3 and 1,800 of potential 10: the first k cuts cost -2, below the
    start of the search for the largest, so i_k is -1 and cluster 0 stands for it, as in the oracle."""
    import paper_1702_04739_amd as iso
    n, m = 6001, 4200
    parent = np.zeros(n, np.int32)
    parent[0] = -1
    length = np.full(n, 1e-9)
    length[0] = 0.0
    p0 = np.full(n, 10.0)
    p0[1:m + 1] = -3.0
    p0[0] = 0.0
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    for k in (m - 50, 3):
        labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k, sigma=1.0, p0=torch.from_numpy(p0).cuda(),
                                                          return_clusters=True)
        lab = labels.cpu().numpy()
        np.testing.assert_array_equal(lab[1:k + 1], np.arange(k))
        assert (lab[k + 1:] == -1).all()
        assert ik == -1.0 and info["jstar"] == 0
        np.testing.assert_allclose((info["cluster_num"] / info["cluster_den"]).cpu().numpy(), -2.0, rtol=1e-6)
