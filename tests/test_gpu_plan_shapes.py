"""A plan's shape and memory as its options change: what csgv_plan_get_opts reports
is what is launched (read from the kernel nodes of a captured launch), handing it
back changes nothing, and a change that does not fit leaves the plan as it was."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

from .test_gpu_decode import P  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def _volume64(P):
    v = np.concatenate([synth.voronoi_u32(64, 20 + 9 * k, seed=k).reshape(-1) for k in range(3)])
    return P.csgv_encode_bricks(v, [6] * 3, 4, origins=np.zeros((3, 3), np.uint32))


def _decode(P, plan, dv, c, ids, lods):
    import torch
    d_ids, d_lods, d_offs, offs, total = dv.tasks(ids, lods)
    n = len(ids)
    out = torch.zeros(total, dtype=torch.int32, device="cuda")
    st = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    plan.launch(None, dv.tensor, d_ids, d_lods, d_offs, n, out, total, st)
    torch.cuda.synchronize()
    want, wst = oracle.decode_tasks(c, ids, lods, offs, total, 4, nthreads=8)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), wst)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want)


class _KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def _hip():
    path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
    hip = ctypes.CDLL(path)
    vp = ctypes.c_void_p
    hip.hipStreamBeginCapture.argtypes = [vp, ctypes.c_int]
    hip.hipStreamEndCapture.argtypes = [vp, ctypes.POINTER(vp)]
    hip.hipGraphGetNodes.argtypes = [vp, vp, ctypes.POINTER(ctypes.c_size_t)]
    hip.hipGraphNodeGetType.argtypes = [vp, ctypes.POINTER(ctypes.c_int)]
    hip.hipGraphKernelNodeGetParams.argtypes = [vp, ctypes.POINTER(_KernelNode)]
    hip.hipGraphDestroy.argtypes = [vp]
    return hip


def _launched(dv, plan, n):
    """(threads, work-groups, LDS bytes) of the decode kernel that a launch of n tasks enqueues."""
    import torch
    hip, stream, graph, count = _hip(), torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    d_ids, d_lods, d_offs, _, total = dv.tasks(np.zeros(n, np.uint32), np.full(n, dv.log2b[0], np.uint8))
    out = torch.zeros(total, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(stream.cuda_stream, 2) == 0
    plan.launch(stream, dv.tensor, d_ids, d_lods, d_offs, n, out, total, None)
    assert hip.hipStreamEndCapture(stream.cuda_stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    found = []
    for node in nodes:
        k = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(k)) == 0
        if k.shared:  # (the binning kernel asks for none)
            found.append((k.block[0], k.grid[0], k.shared))
    assert hip.hipGraphDestroy(graph) == 0
    assert len(found) == 1
    return found[0]


@pytest.mark.parametrize("max_tasks", [5, 300, 512, 513, 600, 3000])
@pytest.mark.parametrize("kw", [{}, dict(wg_size=1024), dict(wg_size=128), dict(lds_slots=8203), dict(wg_size=1024, lds_slots=16384, wgs_per_cu=1)])
def test_the_reported_shape_is_launched_and_may_be_handed_back(P, max_tasks, kw):
    import torch
    dv = P.DeviceVolume(P.encode_volume(synth.voronoi_u32(64, 40, seed=1), 5))
    two = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    plan = P.csgv_plan(dv.info, max_tasks, **kw)
    o = plan.get_opts()
    like = P.csgv_plan(dv.info, max_tasks, wg_size=o.wg_size, lds_slots=o.lds_slots, wgs_per_cu=kw.get("wgs_per_cu", 0))
    shape = _launched(dv, plan, max_tasks)
    assert shape == _launched(dv, like, max_tasks) and shape[0] == o.wg_size
    if kw:
        assert all(getattr(o, k) == v for k, v in kw.items())
    else:
        assert (o.wg_size, o.lds_slots) == ((512, 24576) if max_tasks <= two else (256, 10240))
    if "lds_slots" not in kw and "wg_size" in kw:  # a CU's one work-group of 1024 threads has its LDS to itself
        assert o.lds_slots == (32760 if kw["wg_size"] == 1024 else 10240)
    few = _launched(dv, plan, 5)
    o.sort_tasks = 0  # one change, everything else handed back
    plan.set_opts(**{k: v for k, v in o.as_dict().items() if k != "mode"})
    assert plan.get_opts().as_dict() == o.as_dict()
    assert _launched(dv, plan, max_tasks) == shape and _launched(dv, plan, 5) == few
    plan.set_opts(wg_size=256)  # a choice holds for every number of tasks
    assert _launched(dv, plan, max_tasks)[0] == _launched(dv, plan, 5)[0] == plan.get_opts().wg_size == 256


def test_the_tuner_reports_the_default_shape_of_its_tasks(P):
    # at two tasks per CU and fewer the default is 512 threads with 24,576 slots, which is also the fastest
    # shape where level 5 fits in no smaller split; the time reported for it is then the best one
    import torch
    v = np.concatenate([synth.voronoi_u32(64, 900, seed=k).reshape(-1) for k in range(3)])
    c = P.csgv_encode_bricks(v, [6] * 3, 4, origins=np.zeros((3, 3), np.uint32))
    dv = P.DeviceVolume(c)
    n = 100
    ids, lods = (np.arange(n) % 3).astype(np.uint32), np.ones(n, np.uint8)
    d_ids, d_lods, d_offs, _, total = dv.tasks(ids, lods)
    out = torch.zeros(total, dtype=torch.int32, device="cuda")
    plan = P.csgv_plan(dv.info, n)
    default = plan.get_opts()
    chosen = 0
    for _ in range(5):
        rep = plan.autotune(None, dv.tensor, d_ids, d_lods, d_offs, n, out, total)
        assert 0 < rep.best_ms <= rep.default_ms and rep.tried == 12
        if (rep.chosen.wg_size, rep.chosen.lds_slots) == (default.wg_size, default.lds_slots):
            chosen += 1
            assert rep.default_ms == rep.best_ms
    assert chosen
    assert _launched(dv, plan, n)[0] == rep.chosen.wg_size == plan.get_opts().wg_size
    _decode(P, plan, dv, c, ids, lods)


def test_a_shape_that_does_not_fit_leaves_the_plan_as_it_was(P):
    # 4 million work-groups' scratch is refused by the allocator (5.8 TB)
    c = _volume64(P)
    dv = P.DeviceVolume(c)
    rng = np.random.default_rng(0)
    plan = P.csgv_plan(dv.info, 1 << 22)
    before, few = plan.get_opts().as_dict(), _launched(dv, plan, 40)
    for n in (40, 1500):
        ids, lods = rng.integers(0, 3, n).astype(np.uint32), rng.integers(0, 7, n).astype(np.uint8)
        _decode(P, plan, dv, c, ids, lods)
        with pytest.raises(P.CsgvError) as e:
            plan.set_opts(wgs_per_cu=1 << 14)
        assert e.value.code == P.csgv.CSGV_ENOMEM
        assert plan.get_opts().as_dict() == before and _launched(dv, plan, 40) == few
        _decode(P, plan, dv, c, ids, lods)
    plan.destroy()
    with pytest.raises(P.CsgvError) as e:  # and no plan at all where none fits
        P.csgv_plan(dv.info, 1 << 22, wgs_per_cu=1 << 14)
    assert e.value.code == P.csgv.CSGV_ENOMEM
    _decode(P, P.csgv_plan(dv.info, 40), dv, c, ids[:40], lods[:40])
