"""Captured launches with more tasks than work-groups: the queue's counters, the cost
classes' lists and the packed offsets are set anew by every replay.  New tasks for each
replay, eager launches and other work between them, every replay against the oracle."""
import numpy as np
import pytest

import oracle

from .test_gpu_decode import P, _random_stream_container  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,n,kw", [
    ("plan", 1500, dict(wgs_per_cu=1)),                 # work-groups' lists and single wavefronts' lists
    ("plan", 1500, dict(wgs_per_cu=1, sort_tasks=0)),   # the counter alone
    ("plan", 4500, {}),                                 # the default shape, 18 blocks of the binning kernel
    ("plan", 4500, dict(palette_bits=13)),
    ("noalloc", 4500, {}),                              # control words and table from a kernel before it
    ("noalloc", 200, dict(wg_size=128)),                # no more tasks than work-groups
])
@pytest.mark.parametrize("packed", [True, False])
def test_replays_of_a_queue(P, form, n, kw, packed):
    import torch
    c, Ls = _random_stream_container(77, 40, 4, Ls=(1, 2, 3, 4, 5))
    dv = P.DeviceVolume(c)
    bits = kw.get("palette_bits", 0)
    rng = np.random.default_rng(n)
    L = np.asarray(Ls, np.int64)

    def tasks():
        ids = rng.integers(0, 40, n)
        lods = np.minimum(rng.integers(0, 6, n), L[ids])
        lods[rng.random(n) < 0.4] = 0
        return ids.astype(np.uint32), lods.astype(np.uint8)

    def layout(ids, lods):
        vox = np.int64(1) << (3 * (L[ids.astype(np.int64)] - lods))
        size = P.csgv.paletted_words(vox, bits) if bits else vox
        return (np.cumsum(size) - size).astype(np.uint64), int(size.sum())

    room = 8 * n * 32 ** 3 // (8 if bits else 4)
    d_ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_lods = torch.zeros(n, dtype=torch.uint8, device="cuda")
    d_offs = None if packed else torch.zeros(n, dtype=torch.int64, device="cuda")
    out = torch.zeros(room, dtype=torch.int32, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    plan = P.csgv_plan(dv.info, n, **kw) if form == "plan" else None
    side = torch.cuda.Stream()

    def put(ids, lods, offs):
        d_ids.copy_(torch.from_numpy(ids.view(np.int32)))
        d_lods.copy_(torch.from_numpy(lods))
        if not packed:
            d_offs.copy_(torch.from_numpy(offs.view(np.int64)))

    def launch():
        args = (side, dv.tensor, d_ids, d_lods, d_offs, n, out, room, st)
        if plan:
            plan.launch(*args)
        else:
            P.csgv.csgv_decode_bricks_noalloc(args[0], dv.info, *args[1:], mode=P.MODE_PERSISTENT, **kw)

    def check(what, go):
        ids, lods = tasks()
        offs, total = layout(ids, lods)
        put(ids, lods, offs)
        out[:total + 64].fill_(0x5A5A5A5A)
        st.fill_(-1)
        torch.cuda.synchronize()
        go()
        torch.cuda.synchronize()
        if bits:
            want = np.full(total, 0x5A5A5A5A, np.uint32)
            want, wst = oracle.decode_tasks_paletted(c, ids, lods, offs, total, bits, out=want, nthreads=8)
        else:
            want, wst = oracle.decode_tasks(c, ids, lods, offs, total, 4, nthreads=8, out=np.full(total, 0x5A5A5A5A, np.uint32))
        assert np.array_equal(st.cpu().numpy().view(np.uint32), wst), what
        assert np.array_equal(out[:total].cpu().numpy().view(np.uint32), want), what
        assert int((out[total:total + 64] - 0x5A5A5A5A).abs().sum()) == 0, what  # other work between the replays

    with torch.cuda.stream(side):
        check("eager", launch)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            launch()
        for rep in range(5):
            check("replay %d" % rep, graph.replay)
            if rep == 2:
                check("eager between", launch)
    if plan:
        plan.destroy()
