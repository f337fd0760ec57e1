"""GPU: calls that allocate their own scratch where there is little room.

A memory pool of limited size stands for a device that other programs fill.
A call whose scratch does not fit is refused, and the next one is as before."""
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
