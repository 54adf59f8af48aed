"""The encoder's block-wise operations and multiplied rANS steps against the
oracle's encoder, byte for byte: the six operations of the mask (its bit 6, short
back references, is not one of the oracle encoder's), both neighbour modes,
sides 2..64, palettes that outgrow their first table, every lane count and
coder, and more threads than bricks."""
import numpy as np
import pytest

import oracle


@pytest.fixture(scope="module")
def P():
    import paper_2609_36898_amd  # (not at collection: GPU tests import torch first)
    return paper_2609_36898_amd


def _bricks(rng, lb, l2):
    parts = []
    for k, l in enumerate(l2):
        b = 1 << l
        v = [rng.integers(0, 3, (b,) * 3),                                   # two or three labels: ties of the mode
             rng.integers(0, 1 << 31, (b,) * 3),                             # a palette of every node
             np.where(rng.random((b,) * 3) < 0.03, rng.integers(1, 900, (b,) * 3), 7),
             np.add.outer(np.add.outer(np.arange(b) // 3, np.arange(b) // 5), np.arange(b) // 2),
             np.full((b,) * 3, 5)][k % 5].astype(np.uint64 if lb == 8 else np.uint32)
        if lb == 8:
            v += (v % np.uint64(3)) << np.uint64(40)  # labels that differ above 32 bits only
        parts.append(v.reshape(-1))
    return np.concatenate(parts)


@pytest.mark.parametrize("lb", [4, 8])
@pytest.mark.parametrize("op_mask,nmode", [(63, 0), (63, 1), (0, 0), (1, 0), (14, 1), (30, 0), (48, 0), (62, 1), (59, 0), (55, 1)])
def test_blocks_match_the_oracle(P, lb, op_mask, nmode):
    rng = np.random.default_rng(op_mask + 2 * nmode)
    l2 = [1, 2, 3, 4, 5, 5, 5, 4, 3, 2]
    vox = _bricks(rng, lb, l2)
    for coder in (0, 1, 2):
        kw = dict(origins=np.zeros((len(l2), 3), np.uint32), op_mask=op_mask, neighbor_mode=nmode)
        got = P.csgv_encode_bricks(vox, l2, lb, coder_policy=coder, **kw)
        assert got == oracle.encode_bricks(vox, l2, lb, coder=coder, **kw)


@pytest.mark.parametrize("lane_syms", [1, 16, 63, 300, 5000, 1 << 20])
@pytest.mark.parametrize("n_threads", [1, 3, 64])
def test_lane_counts_match_the_oracle(P, lane_syms, n_threads):
    rng = np.random.default_rng(lane_syms)
    l2 = [5, 6, 2, 1, 4, 5]
    vox = _bricks(rng, 4, l2)
    kw = dict(origins=np.zeros((len(l2), 3), np.uint32), lane_syms=lane_syms)
    got = P.csgv_encode_bricks(vox, l2, 4, coder_policy=2, n_threads=n_threads, **kw)
    assert got == oracle.encode_bricks(vox, l2, 4, coder=2, **kw)
