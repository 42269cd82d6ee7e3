"""Levels of as many blocks as the level passes' tiles change at: one row of 64 per
wave up to 2^18 blocks, two up to 2^21, eight beyond.  The level of the 4-byte blocks
has exactly that many, marked and unmarked ones: copies of 20 bytes hold both pairs of
such blocks, and no two pairs of 8-byte ones."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _text(blocks):
    T = synth.random_text(4 * blocks - 1, 250, blocks)
    rng = np.random.default_rng(blocks)
    for at in rng.integers(T.size // 2, T.size - 40, blocks // 50):
        src = int(rng.integers(0, T.size // 2 - 40))
        T[at:at + 20] = T[src:src + 20]
    return T


@pytest.mark.parametrize("blocks", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 513,
                                    (1 << 21) - 1, 1 << 21, (1 << 21) + 1, (1 << 21) + 2049])
def test_blocks_at_row_switches(blocks):
    torch_cuda()
    import paper_2512_23314_amd as bt
    T = _text(blocks)
    want = oracle.build_tree_par(T, 2, 2)
    L = want.levels[-2]
    assert (L.b, L.c) == (4, blocks) and 0 < L.u < L.c
    ctx = bt.Context(0)
    for kw in ({}, {"lean": True}):
        t = ctx.build(to_device(T), tau=2, leaf_len=2, **kw)
        assert t.level_info(t.height - 1)[1] == blocks
        assert t.serialize() == want.canonical
        t.free()
    ctx.close()
