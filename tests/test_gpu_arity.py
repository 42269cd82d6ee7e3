"""Trees of large arity: the split's two ways to write a block's children, on either
side of arity 64, with children of full and short blocks, in one text and in batches;
and the time of a level with few parents and many children."""
import time

import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [63, 64, 65, 200, 4096])
def test_children(tau):
    torch_cuda()
    import paper_2512_23314_amd as bt
    leaf = 4
    ctx = bt.Context(0)
    texts = []
    for n in (tau * leaf * 3 - 1, tau * leaf * 70 + 5, tau * leaf + 1, 5 * tau * tau // 3 if tau <= 200 else 9 * tau):
        T = np.resize(synth.random_text(n // 3 + 2, 4, n), n)
        T[n // 2::97] ^= 1
        texts.append(T)
    for kw in ({}, {"prune": True}, {"lean": True}):
        want = [oracle.build_tree(T, tau, leaf, prune="prune" in kw).canonical for T in texts]
        for T, w in zip(texts, want):
            t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, **kw)
            assert t.serialize() == w
            t.free()
        off = np.concatenate([[0], np.cumsum([T.size for T in texts])]).astype(np.uint64)
        trees = ctx.build_batch(to_device(np.concatenate(texts)), off, tau=tau, leaf_len=leaf, **kw)
        assert [t.serialize() for t in trees] == want
        bt.free_trees(trees)
    ctx.close()


def test_time_of_many_children():
    """One root block of 2^20 leaves, against the same text with 2^20 root blocks and no
    level below: 136 times as long with a thread per parent, now 8.  The bound lies
    between."""
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    d = to_device(synth.random_text(16 << 20, 4, 3))
    ctx = bt.Context(0)
    ms = []
    for root in (16 << 20, 16):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            t = ctx.build(d, tau=1 << 20, leaf_len=16, root_block_len=root)
            torch.cuda.synchronize()
            best = min(best, 1e3 * (time.perf_counter() - t0))
            t.free()
        ms.append(best)
    ctx.close()
    print("one parent, no parent: %.2f %.2f ms, ratio %.2f" % (ms[0], ms[1], ms[0] / ms[1]))
    assert ms[0] < 40 * ms[1]
