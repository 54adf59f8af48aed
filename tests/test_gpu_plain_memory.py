"""A plain one-shot call where device memory is short: it decodes with the work-groups
whose scratch it gets, down to one; and it asks for no more than the GPU holds.  The
stream-ordered allocations come from a pool of limited size."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

from .test_gpu_decode import P  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

PER_WG_32 = 65536 + 4 * 4096 + (4 * sum(8 ** i for i in range(6)) + 255) // 256 * 256
PER_WG_64 = 65536 + 4 * 32768 + (4 * sum(8 ** i for i in range(7)) + 255) // 256 * 256


class _Props(ctypes.Structure):  # hipMemPoolProps: pinned allocations on device 0
    _fields_ = [("type", ctypes.c_int), ("handles", ctypes.c_int), ("where", ctypes.c_int), ("device", ctypes.c_int),
                ("security", ctypes.c_void_p), ("max_size", ctypes.c_size_t), ("reserved", ctypes.c_ubyte * 56)]


class _Pool:
    """The current device's pool for stream-ordered allocations, with at most `limit` bytes (0: any)."""

    def __init__(self, limit):
        import torch
        self.torch = torch
        torch.zeros(1, device="cuda")
        self.hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
        vp = ctypes.c_void_p
        self.hip.hipMemPoolCreate.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(_Props)]
        self.hip.hipDeviceSetMemPool.argtypes = [ctypes.c_int, vp]
        self.hip.hipDeviceGetDefaultMemPool.argtypes = [ctypes.POINTER(vp), ctypes.c_int]
        self.hip.hipMemPoolGetAttribute.argtypes = [vp, ctypes.c_int, vp]
        self.hip.hipMemPoolDestroy.argtypes = [vp]
        self.pool, self.limit = vp(), limit

    def __enter__(self):
        p = _Props(type=1, where=1, device=0, max_size=self.limit)
        assert self.hip.hipMemPoolCreate(ctypes.byref(self.pool), ctypes.byref(p)) == 0
        assert self.hip.hipDeviceSetMemPool(0, self.pool) == 0
        return self

    def most_used(self):
        v = ctypes.c_uint64()
        assert self.hip.hipMemPoolGetAttribute(self.pool, 8, ctypes.byref(v)) == 0
        return v.value

    def __exit__(self, *a):
        self.torch.cuda.synchronize()
        d = ctypes.c_void_p()
        assert self.hip.hipDeviceGetDefaultMemPool(ctypes.byref(d), 0) == 0
        assert self.hip.hipDeviceSetMemPool(0, d) == 0
        assert self.hip.hipMemPoolDestroy(self.pool) == 0


def _volume64(P):
    rng = np.random.default_rng(1)
    v = [synth.voronoi_u32(64, 20 + 9 * k, seed=k).reshape(-1) for k in range(3)]
    v.append(rng.integers(1, 1 << 30, 64 ** 3).astype(np.uint32))  # chunks, long streams: scratch in use
    return P.csgv_encode_bricks(np.concatenate(v), [6] * 4, 4, origins=np.zeros((4, 3), np.uint32))


def _decode(P, c, ids, lods, dense, **kw):
    import torch
    dv = P.DeviceVolume(c)
    d_ids, d_lods, d_offs, offs, total = dv.tasks(ids, lods)
    n = len(ids)
    out = torch.full((total,), 7, dtype=torch.int32, device="cuda")
    st = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    P.csgv_decode_bricks(None, dv.info, dv.tensor, d_ids, d_lods, None if dense else d_offs, n, out, total, st, **kw)
    torch.cuda.synchronize()
    want, wst = oracle.decode_tasks(c, ids, lods, offs, total, 4, nthreads=8)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), wst)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("room", [1, 2, 5, 40])
@pytest.mark.parametrize("n", [90, 600])
def test_plain_calls_make_do_with_less_scratch(P, n, room, dense):
    c = _volume64(P)
    rng = np.random.default_rng(n)
    ids, lods = rng.integers(0, 4, n).astype(np.uint32), rng.integers(1, 7, n).astype(np.uint8)
    lods[:8] = 0
    limit = room * PER_WG_64 + (64 << 10)
    for kw in ({}, dict(mode=0, wg_size=256)):
        with _Pool(limit) as pool:  # (one for each call: memory given back still counts)
            _decode(P, c, ids, lods, dense, **kw)
            assert PER_WG_64 <= pool.most_used() <= limit
    with _Pool(limit):
        with pytest.raises(P.CsgvError):  # the persistent form is refused, as ever
            _decode(P, c, ids, lods, dense, mode=P.MODE_PERSISTENT)
        _decode(P, c, ids, lods, dense)  # and leaves no error to the next call


def test_plain_calls_take_scratch_for_resident_work_groups(P):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    c = P.encode_volume(synth.voronoi_u32(64, 40, seed=1), 5)
    n = 6000
    ids, lods = (np.arange(n) % 8).astype(np.uint32), np.full(n, 4, np.uint8)
    with _Pool(0) as pool:
        _decode(P, c, ids, lods, False, mode=0, wgs_per_cu=1000)
        assert pool.most_used() <= 4 * cus * PER_WG_32 + 64 * n + (4 << 20)
