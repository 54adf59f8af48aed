"""GPU parity on the edges between the decoder's paths: cubes decoded by single
wavefronts, by work-groups in LDS or in chunks, streams that do and do not fit in
LDS, the binning kernel's blocks, launch shapes, unaligned outputs and packed
palette indices.  Everything is compared with the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
import synth

from .test_gpu_decode import P, _compare, _random_stream_container, _say  # noqa: F401  (P is a fixture)
from .test_gpu_paletted import _compare as _compare_paletted

pytestmark = pytest.mark.gpu


def _run(P, c, ids, lods, dense=True, shift=0, **kw):
    """One decode; (labels, status, offsets).  shift: elements before the first task's output."""
    import torch
    dv = P.DeviceVolume(c)
    ids, lods = np.asarray(ids, np.uint32), np.asarray(lods, np.uint8)
    l2 = P.brick_log2b(c)[np.minimum(ids, dv.info.n_bricks - 1).astype(np.int64)].astype(np.int64)
    named = (ids < dv.info.n_bricks) & (lods <= l2)
    size = np.where(named, np.int64(1) << (3 * np.maximum(l2 - lods, 0)), 0)
    offs = (np.cumsum(size) - size + shift).astype(np.uint64)
    total = int(size.sum()) + shift + 1
    out = torch.full((total,), 0x5A5A5A5A, dtype=dv.dtype, device="cuda")
    st = torch.full((len(ids),), -1, dtype=torch.int32, device="cuda")
    P.csgv_decode_bricks(None, dv.info, dv.tensor, torch.from_numpy(ids.view(np.int32)).cuda(), torch.from_numpy(lods).cuda(),
                         None if dense else torch.from_numpy(offs.view(np.int64)).cuda(), len(ids), out, total, st, **kw)
    torch.cuda.synchronize()
    ut = np.uint64 if dv.info.label_bytes == 8 else np.uint32
    want, wst = oracle.decode_tasks(c, ids, lods, offs, total, int(dv.info.label_bytes), nthreads=8,
                                    out=np.full(total, 0x5A5A5A5A, ut))
    return out.cpu().numpy().view(ut), st.cpu().numpy().view(np.uint32), want, wst


def _same(got):
    out, st, want, wst = got
    assert np.array_equal(st, wst), np.nonzero(st != wst)[0][:10]
    assert np.array_equal(out, want), np.nonzero(out != want)[0][:10]
    return wst


@pytest.mark.parametrize("n", [1, 4, 5, 17, 1025, 4099])
@pytest.mark.parametrize("lb", [4, 8])
def test_small_cubes_by_single_wavefronts(P, n, lb):
    # sides 1..8 among some larger ones, every coder and lane count, damaged records
    c, Ls = _random_stream_container(50 + lb, 30, lb, Ls=(1, 2, 3, 5))
    offs = oracle.brick_offsets(c)
    rng = np.random.default_rng(n)
    c = bytearray(c)
    for k in range(0, 30, 7):
        c[int(rng.integers(offs[k], offs[k + 1]))] ^= 1 << int(rng.integers(8))
    c = bytes(c)
    ids = rng.integers(0, 30, n)
    L = np.asarray(Ls)[ids]
    lods = np.where((L == 5) & (rng.random(n) < 0.9), 2 + rng.integers(0, 4, n), rng.integers(0, L + 1))
    _compare(P, c, ids, lods, modes=(2,))


@pytest.mark.parametrize("n", [255, 256, 257, 777])
@pytest.mark.parametrize("sort", [0, 1])
def test_dense_offsets_over_blocks_of_tasks(P, n, sort):
    # the offsets of a launch without them; tasks that name no brick or LOD take no room
    c = P.encode_volume(synth.voronoi_voids(128, 312, seed=3), 5)
    rng = np.random.default_rng(n)
    ids, lods = rng.integers(0, 64, n), rng.integers(2, 6, n)
    ids[::50], lods[7::60] = 64 + np.arange(len(ids[::50])), 6
    for mode in (0, 2):
        st = _same(_run(P, c, ids, lods, mode=mode, sort_tasks=sort))
        assert (st == 1).any()


@pytest.mark.parametrize("mode,kw", [(0, {}), (2, dict(sort_tasks=0)), (2, dict(sort_tasks=1)), (2, dict(wg_size=512)), (2, dict(wg_size=1024))])
def test_more_tasks_than_work_groups(P, mode, kw):
    c = P.encode_volume(synth.voronoi_voids(128, 312, seed=3), 5)
    rng = np.random.default_rng(1)
    _same(_run(P, c, rng.integers(0, 64, 1500), rng.integers(0, 4, 1500), mode=mode, wgs_per_cu=1, **kw))


@pytest.mark.parametrize("n", [511, 512, 513])
def test_default_shape_at_two_tasks_per_cu(P, n):
    c = P.encode_volume(synth.voronoi_voids(128, 312, seed=3), 5)
    _same(_run(P, c, np.arange(n) % 64, np.arange(n) // 64 % 3, mode=2))


@pytest.mark.parametrize("lane_syms", [16, 48, 200, 900, 4000, 1 << 20])
@pytest.mark.parametrize("kw", [{}, dict(lds_slots=8192), dict(wg_size=512, lds_slots=32760)])
def test_lane_counts_and_streams_that_fit_or_not(P, lane_syms, kw):
    # 256 lanes down to one; smooth bricks whose words fit in LDS, noise whose words do not,
    # and a level 5 that outgrows the slot area
    v = synth.voronoi_u32(64, 40, seed=4)
    rng = np.random.default_rng(2)
    v[:32, :32, :32] = rng.integers(1, 20, (32, 32, 32))
    v[32:, :32, :32] = rng.integers(1, 3, (32, 32, 32))
    v[:32, 32:, :32] = np.where(rng.random((32, 32, 32)) < 0.07, 9, v[:32, 32:, :32])
    c = P.encode_volume(v, 5, coder_policy=2, lane_syms=lane_syms)
    _compare(P, c, np.repeat(np.arange(8), 3), np.tile([0, 1, 2], 8), modes=(2,), **kw)


@pytest.mark.parametrize("lane_syms", [16, 900, 1 << 20])
@pytest.mark.parametrize("kw", [{}, dict(wg_size=256, lds_slots=8192), dict(wg_size=1024)])
def test_64_bricks_in_chunks(P, lane_syms, kw):
    # smooth, noisy and palette-only 64^3 bricks: implied and explicit level-5 nodes, long delta chains
    rng = np.random.default_rng(3)
    smooth = synth.voronoi_u32(64, 30, seed=5)
    half = smooth.copy()
    half[:, :, 32:] = rng.integers(1, 500, (64, 64, 32))
    noise = rng.integers(1, 1 << 30, (64, 64, 64)).astype(np.uint32)
    bricks = np.concatenate([smooth.reshape(-1), half.reshape(-1), noise.reshape(-1)])
    c = P.csgv_encode_bricks(bricks, [6, 6, 6], 4, origins=np.zeros((3, 3), np.uint32), lane_syms=lane_syms)
    _compare(P, c, np.repeat(np.arange(3), 3), np.tile([0, 1, 2], 3), modes=(2,), **kw)


@pytest.mark.parametrize("lb", [4, 8])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_outputs(P, lb, shift):
    v = synth.voronoi_small(0).astype(np.uint64 if lb == 8 else np.uint32)
    c = P.encode_volume(v, 5)
    n = 64
    for mode in (0, 2):
        _same(_run(P, c, np.arange(n), np.arange(n) % 6, dense=False, shift=shift, mode=mode))


@pytest.mark.parametrize("bits", [6, 7, 10, 12, 16, 17])
@pytest.mark.parametrize("kw", [{}, dict(wg_size=512), dict(wg_size=1024, lds_slots=8192), dict(wg_size=1024, lds_slots=32760)])
def test_paletted_words_across_rows(P, bits, kw):
    # 3 bits up to one voxel a word; words that straddle the 512 voxels a wavefront
    # packs at a time, level 5 in LDS with and without room for them
    v = synth.voronoi_u32(64, 40, seed=4)
    rng = np.random.default_rng(2)
    v[32:, 32:, 32:] = np.where(rng.random((32, 32, 32)) < 0.02, 99, v[32:, 32:, 32:])
    v[:32, :32, :32] = np.where(rng.random((32, 32, 32)) < 0.038, 99, v[:32, :32, :32])
    c = P.encode_volume(v, 5)
    st = _compare_paletted(P, c, np.repeat(np.arange(8), 3), np.tile([0, 1, 2], 8), bits, modes=(2,), **kw)
    assert (st == 0).all()


@pytest.mark.parametrize("bits", [1, 2, 3, 5, 16])
def test_paletted_levels_in_chunks_and_narrow_indices(P, bits):
    # few labels per brick in noise: level 5 in chunks; 16 bits: more than 32768 palette entries
    rng = np.random.default_rng(4)
    if bits < 16:
        b, kw = rng.integers(1, 1 + (1 << bits), (2, 32, 32, 32)).astype(np.uint32), {}
    else:
        b, kw = synth.test_brick_u64(32, 0, 1 << 30, base=1, seed=9).astype(np.uint32)[None], dict(op_mask=0)
    c = P.csgv_encode_bricks(b.reshape(-1), [5] * len(b), 4, origins=np.zeros((len(b), 3), np.uint32), **kw)
    ids, lods = np.repeat(np.arange(len(b)), 3), np.tile([0, 1, 2], len(b))
    _compare_paletted(P, c, ids, lods, bits)


def test_captured_launches_replay(P):
    import torch
    c = P.encode_volume(synth.voronoi_voids(128, 312, seed=8), 5)
    dv = P.DeviceVolume(c)
    n = 300
    rng = np.random.default_rng(0)
    sets = [(rng.integers(0, 64, n), np.sort(rng.integers(0, 6, n))) for _ in range(3)]
    sets = [(i, sets[0][1]) for i, _ in sets]  # the same sizes: one output layout
    d_ids, d_lods, d_offs, offs, total = dv.tasks(*sets[0])
    out = torch.zeros(total, dtype=torch.int32, device="cuda")
    st = torch.zeros(n, dtype=torch.int32, device="cuda")
    plan = P.csgv_plan(dv.info, n)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        plan.launch(side.cuda_stream, dv.tensor, d_ids, d_lods, d_offs, n, out, total, st)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            plan.launch(side.cuda_stream, dv.tensor, d_ids, d_lods, d_offs, n, out, total, st)
    for rep in range(6):
        ids, lods = sets[rep % 3]
        d_ids.copy_(torch.from_numpy(np.asarray(ids, np.uint32).view(np.int32)))
        out.zero_()
        st.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want, wst = oracle.decode_tasks(c, ids, lods, offs, total, 4, nthreads=8)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), wst), rep
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want), rep
        assert int((out.float() * 0.5).sum() > 0)  # other work between the replays
    plan.destroy()


@pytest.mark.parametrize("lane_syms", [16, 64, 300])
@pytest.mark.parametrize("lb", [4, 8])
def test_long_streams_at_the_end_of_the_container(P, lane_syms, lb):
    # containers whose only record's words do not fit in LDS: their last words are the file's last bytes
    for seed in range(8):
        rng = np.random.default_rng(seed)
        b = rng.integers(1, 20 + 5 * seed, (32, 32, 32)).astype(np.uint64 if lb == 8 else np.uint32)
        c = P.csgv_encode_bricks(b.reshape(-1), [5], lb, origins=np.zeros((1, 3), np.uint32), coder_policy=2, lane_syms=lane_syms)
        want, st = _compare(P, c, [0], [0], modes=(0, 2))
        assert st[0] == 0


@pytest.mark.parametrize("sort", [0, 1])
@pytest.mark.parametrize("dense", [True, False])
def test_queue_of_one_block_without_a_plan(P, sort, dense):
    # more tasks than the fixed scratch has work-groups for 64^3 bricks, few enough for one block of
    # the binning kernel, which then also sets the control words and the table; and larger calls between
    import torch
    b = np.concatenate([synth.voronoi_u32(64, 20 + 9 * k, seed=k).reshape(-1) for k in range(4)])
    c = P.csgv_encode_bricks(b, [6] * 4, 4, origins=np.zeros((4, 3), np.uint32))
    dv = P.DeviceVolume(c)
    rng = np.random.default_rng(5)
    for n in (130, 256, 600, 91, 256, 3):
        ids, lods = rng.integers(0, 4, n).astype(np.uint32), rng.integers(1, 7, n).astype(np.uint8)
        lods[: n // 50] = 0
        d_ids, d_lods, d_offs, offs, total = dv.tasks(ids, lods)
        out = torch.zeros(total, dtype=torch.int32, device="cuda")
        st = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        P.csgv.csgv_decode_bricks_noalloc(None, dv.info, dv.tensor, d_ids, d_lods, None if dense else d_offs, n, out, total, st,
                                          mode=P.MODE_PERSISTENT, sort_tasks=sort)
        torch.cuda.synchronize()
        want, wst = oracle.decode_tasks(c, ids, lods, offs, total, 4, nthreads=8)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), wst), n
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want), n
