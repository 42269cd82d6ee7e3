"""Texts with many root blocks (s_hint, a small root_block_len): the blocks of texts
that enter a level, one or many of them, of 1 block up to more than a launch's
threads take at once, and the time that takes."""
import time

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 63, 64, 65, 255, 1025, 4097, 1050001])
def test_root_blocks(blocks):
    torch_cuda()
    import paper_2512_23314_amd as bt
    tau, leaf = 2, 4
    ctx = bt.Context(0)
    for b1 in (leaf, 2 * leaf):
        T = np.resize(synth.random_text(min(blocks * b1, 70003), 4, blocks), blocks * b1 - b1 // 2)
        t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, root_block_len=b1)
        assert t.level_info(1)[1] == blocks
        assert t.serialize() == oracle.build_tree_par(T, tau, leaf, b1=b1).canonical
        t.free()
    ctx.close()


@pytest.mark.parametrize("count,most", [(1, 70000), (3, 70000), (40, 3000), (5000, 64), (5000, 65)])
def test_root_blocks_of_batches(count, most):
    torch_cuda()
    import paper_2512_23314_amd as bt
    tau, leaf, b1 = 2, 4, 8
    rng = np.random.default_rng(most)
    sizes = rng.integers(0, most * b1 + 1, count) // rng.choice([1, 30], count)
    sizes[-1] = most * b1 - 3
    texts = [synth.random_text(int(n), 3, i) for i, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    ctx = bt.Context(0)
    d = to_device(np.concatenate(texts))
    for kw, root in (({"root_block_len": b1}, b1), ({"s_hint": 300}, None)):
        trees = ctx.build_batch(d, off, tau=tau, leaf_len=leaf, **kw)
        for k in list(range(0, count, max(1, count // 60))) + [count - 1]:
            want = oracle.build_tree_par(texts[k], tau, leaf, **({"b1": root} if root else {"s_hint": 300}))
            assert trees[k].serialize() == want.canonical
        bt.free_trees(trees)
    ctx.close()


def test_time_of_root_blocks():
    """A text of 2^24 root blocks that are its leaves, against 2^18 of them: 11 times
    as long when one workgroup wrote them, now 1.5.  The bound lies between."""
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    d = to_device(synth.random_text(64 << 20, 4, 3))
    ctx = bt.Context(0)
    ms = []
    for leaf in (4, 256):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            t = ctx.build(d, tau=2, leaf_len=leaf, root_block_len=leaf)
            torch.cuda.synchronize()
            best = min(best, 1e3 * (time.perf_counter() - t0))
            t.free()
        ms.append(best)
    ctx.close()
    print("2^24, 2^18 root blocks: %.2f %.2f ms, ratio %.2f" % (ms[0], ms[1], ms[0] / ms[1]))
    assert ms[0] < 4 * ms[1]
