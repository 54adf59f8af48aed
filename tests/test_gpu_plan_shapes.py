"""A plan's shape and memory as its options change: a change that does not fit
leaves the plan as it was."""
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


def test_a_shape_that_does_not_fit_leaves_the_plan_as_it_was(P):
    # 4 million work-groups' scratch is refused by the allocator (5.8 TB)
    c = _volume64(P)
    dv = P.DeviceVolume(c)
    rng = np.random.default_rng(0)
    plan = P.csgv_plan(dv.info, 1 << 22)
    before = plan.get_opts().as_dict()
    for n in (40, 1500):
        ids, lods = rng.integers(0, 3, n).astype(np.uint32), rng.integers(0, 7, n).astype(np.uint8)
        _decode(P, plan, dv, c, ids, lods)
        with pytest.raises(P.CsgvError) as e:
            plan.set_opts(wgs_per_cu=1 << 14)
        assert e.value.code == P.csgv.CSGV_ENOMEM
        assert plan.get_opts().as_dict() == before
        _decode(P, plan, dv, c, ids, lods)
    plan.destroy()
    with pytest.raises(P.CsgvError) as e:  # and no plan at all where none fits
        P.csgv_plan(dv.info, 1 << 22, wgs_per_cu=1 << 14)
    assert e.value.code == P.csgv.CSGV_ENOMEM
    _decode(P, P.csgv_plan(dv.info, 40), dv, c, ids[:40], lods[:40])
