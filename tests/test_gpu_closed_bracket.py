"""GPU: brackets of Algorithm 2 that are closed from the start.

With potentials below zero the printed lower end (phi_* + p_*) / omega^* can
exceed the upper end (phi^* + p^*) / omega_*, so that no midpoint lies between
them and the subpartition is the decision at the upper end.  Every k of the
all-k sweep then records in its own pass.  The tree is a path of equal edges
with one potential, just below the mean flow, at every vertex (the vertices of
a regular simplex have equal sums of distances), in one piece of the tree walk
and in several.  Against the FP64 oracle: labels equal, i_k within 1e-12.
"""
import numpy as np
import pytest

from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bracket", ["pow2", "paper"])
@pytest.mark.parametrize("n,eps", [(40, 1e-6), (200, 1e-8), (1200, 1e-10)])
def test_closed_bracket_all_k(orc, n, eps, bracket):
    import paper_1702_04739_amd as iso
    parent = np.arange(-1, n - 1, dtype=np.int32)
    length = np.ones(n)
    length[0] = 0.0
    X = np.eye(n, dtype=np.float32)
    flow = np.exp(-1.0)
    alpha = flow * (n - 1) / n * (1.0 - eps) / ((n - 1) * np.sqrt(2.0))
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    p0 = -iso.graph_weights(torch.from_numpy(X).cuda(), 1.0, alpha=alpha, omega=False)[1]
    kmax = 12
    H.log("closed bracket n=%d %s" % (n, bracket))
    ik_all, lab_all, _ = iso.subpartition_all_k(pg, lg, kmax, sigma=1.0, bracket=bracket, p0=p0)
    for k in range(2, kmax + 1):
        ref = orc.subpartition(parent, length, k, sigma=1.0, bracket=bracket, alpha_pot=-alpha, X=X)
        assert ref.iters == 0 and ref.alpha0 >= ref.beta0
        labels, ik, info = iso.isoperimetric_subpartition(pg, lg, k, sigma=1.0, bracket=bracket, p0=p0)
        assert info["iters"] == 0
        np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
        np.testing.assert_array_equal(lab_all[k - 2].cpu().numpy(), ref.labels)
        assert abs(ik - ref.i_k) <= 1e-12 * abs(ref.i_k) and ik_all[k - 2] == ik


def test_weights_that_are_no_numbers_are_refused():
    """A NaN weight makes the printed lower end NaN: no bracket, hence an error and no labels, for one k and for all."""
    import paper_1702_04739_amd as iso
    n = 60
    parent = np.arange(-1, n - 1, dtype=np.int32)
    length = np.ones(n)
    length[0] = 0.0
    om = np.ones(n)
    om[n // 2] = np.nan
    pg, lg = torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda()
    kw = dict(sigma=1.0, bracket="paper", omega0=torch.from_numpy(om).cuda())
    with pytest.raises(iso._lib.IsoError):
        iso.isoperimetric_subpartition(pg, lg, 3, **kw)
    with pytest.raises(iso._lib.IsoError):
        iso.subpartition_all_k(pg, lg, 4, **kw)
