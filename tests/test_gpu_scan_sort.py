"""GPU: the prefix sums and the radix sort under the tree stage and the rooting,
at the sizes where they change form: one, four and eight steps per wave, one
pass of a workgroup and two, many workgroups (above 65,536 elements), four and
sixteen keys per thread (262,144 keys).  The child lists, and with them the
partition, come from the sort and the scan of its digit counts: labels and
cluster sizes against the FP64 oracle, i_k to 1e-12 (the device's and the host's
exp differ by an ulp).  The rooting scans the degrees: a tree along a line has a
known parent for every vertex."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [4096, 4097, 16383, 32769, 65536, 65537, 131073, 262144, 262145])
def test_child_lists_at_size(orc, n):
    import paper_1702_04739_amd as iso
    rng = np.random.default_rng(n)
    parent = np.concatenate([[-1], rng.integers(0, np.arange(1, n))]).astype(np.int32)
    length = rng.lognormal(0.0, 0.5, n)
    length[0] = 0.0
    ref = orc.subpartition(parent, length, 3)
    labels, ik, info = iso.isoperimetric_subpartition(torch.from_numpy(parent).cuda(), torch.from_numpy(length).cuda(), 3,
                                                      return_clusters=True)
    assert abs(ik - ref.i_k) <= 1e-12 * ref.i_k
    np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
    np.testing.assert_array_equal(info["cluster_size"].cpu().numpy(), ref.cl_size)


@pytest.mark.parametrize("n", [4097, 16383, 32768, 65535, 65536, 65537, 73729])
def test_rooting_at_size(n):
    """Points at distinct places along a line, in random order: every vertex's
    parent is its neighbour on the side of vertex 0."""
    import paper_1702_04739_amd as iso
    place = np.random.default_rng(n).permutation(n)
    X = torch.from_numpy(place.astype(np.float32)[:, None]).cuda()
    parent, length, _ = iso.mst(X)
    at = np.empty(n, np.int64)
    at[place] = np.arange(n)
    step = np.sign(place[0] - place)
    want = np.where(step == 0, -1, at[np.clip(place + step, 0, n - 1)])
    np.testing.assert_array_equal(parent.cpu().numpy(), want)
    np.testing.assert_array_equal(length.cpu().numpy(), (step != 0).astype(np.float64))
