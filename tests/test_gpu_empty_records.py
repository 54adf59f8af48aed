"""Records without a symbol: every level's end is 0, so the place of the first
symbol, which decides the verdict of level 0, holds none.  GPU against the CPU
oracle, in the forms that keep symbols in LDS, in scratch and in the record."""
import numpy as np
import pytest

import synth
from oracle import brick_offsets

from .test_gpu_decode import P, _compare  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coder", [1, 2])
@pytest.mark.parametrize("lane_syms", [64, 1 << 20])
@pytest.mark.parametrize("kw", [{}, dict(wg_size=256, lds_slots=8192), dict(wg_size=1024, lds_slots=32760)])
def test_records_without_symbols(P, coder, lane_syms, kw):
    for l2 in (5, 6):
        side = 1 << l2
        v = np.concatenate([synth.voronoi_u32(side, 30 + k, seed=k).reshape(-1) for k in range(4)])
        c = bytearray(P.csgv_encode_bricks(v, [l2] * 4, 4, origins=np.zeros((4, 3), np.uint32), coder_policy=coder,
                                           lane_syms=lane_syms))
        offs = brick_offsets(bytes(c))
        for k in (0, 2):  # (sound records between them)
            at = int(offs[k]) + 8
            c[at:at + 4 * (l2 + 1)] = bytes(4 * (l2 + 1))
        ids, lods = np.repeat(np.arange(4), l2 + 1), np.tile(np.arange(l2 + 1), 4)
        _, st = _compare(P, bytes(c), ids, lods, **kw)
        assert (st[(ids == 0) | (ids == 2)] == 2).all() and (st[(ids == 1) | (ids == 3)] == 0).all()
        _compare(P, bytes(c), np.tile(ids, 60), np.tile(lods, 60), modes=(2,), wgs_per_cu=1, **kw)
