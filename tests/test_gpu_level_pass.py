"""The level passes' one-launch prefix sums at the edges of their tiles (256, 512
and 2048 elements by the level's size): levels of 1 to 2^21 + 1 blocks, batches of 1 to 2049 texts, and empty
texts that enter a level with the others (root_block_len)."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_same_tree, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 63, 64, 65, 2047, 2048, 2049, 4096, 4097])
def test_blocks_at_tile_edges(blocks):
    torch_cuda()
    import paper_2512_23314_amd as bt
    leaf, tau = 8, 2
    ctx = bt.Context(0)
    for tail in (0, 5):
        n = blocks * leaf * tau - (leaf * tau - tail if tail else 0)
        if n <= 0:
            continue
        for T in (synth.random_text(n, 4, blocks), synth.random_text(n, 200, blocks),
                  synth.periodic_text(n, max(1, n // 3), blocks)):
            for kw in ({}, {"prune": True}, {"rank_select": True}):
                t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, **kw)
                want = oracle.build_tree(T, tau, leaf, prune=bool(kw.get("prune")))
                assert_same_tree(t, want)
                t.free()
    ctx.close()


@pytest.mark.parametrize("count", [1, 2, 2047, 2048, 2049])
def test_texts_at_tile_edges(count):
    torch_cuda()
    import paper_2512_23314_amd as bt
    tau, leaf, root = 2, 4, 16
    rng = np.random.default_rng(count)
    sizes = rng.integers(0, 90, count)
    sizes[rng.integers(0, count, max(1, count // 5))] = 0
    sizes[-1] = 0
    texts = [synth.random_text(int(n), 2, i) for i, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    ctx = bt.Context(0)
    cat = np.concatenate(texts + [np.zeros(1, np.uint8)])
    for kw, b1 in (({"root_block_len": root}, root), ({}, None)):
        trees = ctx.build_batch(to_device(cat), off, tau=tau, leaf_len=leaf, **kw)
        for T, t in zip(texts, trees):
            assert t.serialize() == oracle.build_tree(T, tau, leaf, b1=b1).canonical
        bt.free_trees(trees)
    ctx.close()


@pytest.mark.parametrize("blocks", [255, 256, 257, 511, 65537, (1 << 18) - 1, (1 << 18) + 1, (1 << 21) - 3, (1 << 21) + 1])
def test_blocks_at_row_edges(blocks):
    torch_cuda()
    import paper_2512_23314_amd as bt
    T = synth.random_text(4 * blocks - 1, 250, blocks)
    T[blocks:blocks + blocks // 3] = T[:blocks // 3]
    ctx = bt.Context(0)
    t = ctx.build(to_device(T), tau=2, leaf_len=2)
    assert t.serialize() == oracle.build_tree_par(T, 2, 2).canonical
    t.free()
    ctx.close()
