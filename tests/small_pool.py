"""A stream-ordered allocator pool of a given size in place of the device's, for
tests of what a call does with little workspace (torch's own memory is not taken
from it)."""
import contextlib
import ctypes


class _Location(ctypes.Structure):
    _fields_ = [("type", ctypes.c_int), ("id", ctypes.c_int)]


class _Props(ctypes.Structure):  # hipMemPoolProps
    _fields_ = [("allocType", ctypes.c_int), ("handleTypes", ctypes.c_int), ("location", _Location),
                ("security", ctypes.c_void_p), ("maxSize", ctypes.c_size_t), ("reserved", ctypes.c_ubyte * 56)]


@contextlib.contextmanager
def small_pool(megabytes):
    import torch
    torch.cuda.synchronize()
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    pool, old = ctypes.c_void_p(), ctypes.c_void_p()
    props = _Props(allocType=1, location=_Location(1, 0), maxSize=megabytes << 20)
    assert hip.hipDeviceGetMemPool(ctypes.byref(old), 0) == 0
    assert hip.hipMemPoolCreate(ctypes.byref(pool), ctypes.byref(props)) == 0
    assert hip.hipDeviceSetMemPool(0, pool) == 0
    try:
        yield
        torch.cuda.synchronize()
    finally:
        assert hip.hipDeviceSetMemPool(0, old) == 0
        assert hip.hipMemPoolDestroy(pool) == 0
