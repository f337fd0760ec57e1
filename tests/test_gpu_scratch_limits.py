"""GPU: calls that allocate their own scratch where there is little room.

A memory pool of limited size stands for a device that other programs fill.
The tree of few points takes the screened rounds where the distance matrix does
not fit, and the full-graph weights take smaller blocks; the results are the
ones with room, bit for bit.  Where even that does not fit: out of memory, and
the next call is as before."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


class _PoolProps(ctypes.Structure):
    _fields_ = [("allocType", ctypes.c_int), ("handleTypes", ctypes.c_int), ("locType", ctypes.c_int),
                ("locId", ctypes.c_int), ("security", ctypes.c_void_p), ("maxSize", ctypes.c_size_t),
                ("reserved", ctypes.c_ubyte * 56)]


class _Room:
    """The device's stream-ordered allocations limited to `bytes` in all."""

    def __init__(self, limit):
        self.limit = limit

    def __enter__(self):
        torch.cuda.synchronize()
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.dev = torch.cuda.current_device()
        self.pool, self.old = ctypes.c_void_p(), ctypes.c_void_p()
        props = _PoolProps(1, 0, 1, self.dev, None, self.limit)
        assert self.hip.hipDeviceGetMemPool(ctypes.byref(self.old), self.dev) == 0
        assert self.hip.hipMemPoolCreate(ctypes.byref(self.pool), ctypes.byref(props)) == 0
        assert self.hip.hipDeviceSetMemPool(self.dev, self.pool) == 0
        return self

    def __exit__(self, *exc):
        torch.cuda.synchronize()
        assert self.hip.hipDeviceSetMemPool(self.dev, self.old) == 0
        assert self.hip.hipMemPoolDestroy(self.pool) == 0


def _mst(X, recheck):
    """iso_mst with its own workspace: (parent, length, info)."""
    from paper_1702_04739_amd import _lib
    lib = _lib.load()
    n, d = X.shape
    parent = torch.empty(n, dtype=torch.int32, device="cuda")
    length = torch.empty(n, dtype=torch.float64, device="cuda")
    info = _lib.MstInfo()
    rc = lib.iso_mst(ctypes.c_void_p(X.data_ptr()), n, d, d, _lib.PRECISION["fp32"], _lib.RECHECK[recheck], 0,
                     ctypes.c_void_p(parent.data_ptr()), ctypes.c_void_p(length.data_ptr()), ctypes.byref(info), None, 0,
                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    _lib.check(rc, "iso_mst")
    torch.cuda.synchronize()
    return parent.cpu().numpy(), length.cpu().numpy(), info


def test_a_refused_call_leaves_no_error_behind():
    from paper_1702_04739_amd._lib import IsoError
    X = torch.from_numpy(np.random.default_rng(2).standard_normal((5000, 16)).astype(np.float32)).cuda()
    p0, l0, _ = _mst(X, "fp32")
    with _Room(16 << 20), pytest.raises(IsoError):
        _mst(X, "fp32")
    p1, l1, _ = _mst(X, "fp32")
    np.testing.assert_array_equal(p1, p0)
    np.testing.assert_array_equal(l1, l0)


@pytest.mark.parametrize("recheck", ["fp32", "fp64"])
def test_tree_without_room_for_the_matrix(recheck):
    from paper_1702_04739_amd._lib import IsoError
    X = torch.from_numpy(np.random.default_rng(1).standard_normal((4096, 16)).astype(np.float32)).cuda()
    p0, l0, i0 = _mst(X, recheck)
    assert i0.tile_pairs == 0
    with _Room(60 << 20):
        p1, l1, i1 = _mst(X, recheck)
    assert i1.tile_pairs > 0
    np.testing.assert_array_equal(p1, p0)
    np.testing.assert_array_equal(l1, l0)
    with _Room(16 << 20), pytest.raises(IsoError):
        _mst(X, recheck)
    p2, l2, i2 = _mst(X, recheck)
    assert i2.tile_pairs == 0
    np.testing.assert_array_equal(p2, p0)


@pytest.mark.parametrize("n,limit", [(2000, 24 << 20), (5000, 24 << 20), (777, 1 << 20)])
def test_graph_weights_in_smaller_blocks(n, limit):
    import paper_1702_04739_amd as iso
    X = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 9)).astype(np.float32)).cuda()
    om0, p0 = iso.graph_weights(X, 1.3, alpha=0.05)
    with _Room(limit):
        om1, p1 = iso.graph_weights(X, 1.3, alpha=0.05)
        torch.cuda.synchronize()
    assert torch.equal(om1, om0) and torch.equal(p1, p0)


def test_tree_where_torch_has_no_room():
    """torch's allocator, which the Python call asks first, limited to 40 MiB beyond what it holds."""
    import paper_1702_04739_amd as iso
    X = torch.from_numpy(np.random.default_rng(3).standard_normal((4096, 16)).astype(np.float32)).cuda()
    p0, l0, i0 = iso.mst(X)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(X.device).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (40 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(134 << 20, dtype=torch.uint8, device="cuda")
        with _Room(60 << 20):
            p1, l1, i1 = iso.mst(X)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert i0["tile_pairs"] == 0 and i1["tile_pairs"] > 0
    assert torch.equal(p1, p0) and torch.equal(l1, l0)
