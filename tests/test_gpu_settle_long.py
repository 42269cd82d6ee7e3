"""Verification of keys compared in chunks: two to five chunks of 4 KiB (weak
fingerprints: most fail, in any chunk), and keys past 8 MiB, whose chunks grow.
Every key of the periodic texts occurs earlier, at any alignment, but for the changed
bytes and the short final keys."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_same_tree, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [2049, 4096, 5000, 8193])
def test_chunks(leaf):
    torch_cuda()
    import paper_2512_23314_amd as bt
    ctx = bt.Context(0)
    b = 2 * leaf
    for n, step in ((40 * b + leaf // 2 + 1, 0), (40 * b, 7), (61 * b + 3, 5)):
        T = np.resize(synth.random_text(5 * b + 7, 4, leaf), n)
        if step:  # changed bytes at every place of a chunk, so that some keys are new
            T[np.arange(3 * b, n, step * b + 1025)] ^= 1
        want = oracle.build_tree(T, 2, leaf)
        for flags in (0, bt.BT_DBG_WEAK_HASH):
            t = ctx.build(to_device(T), tau=2, leaf_len=leaf, debug_flags=flags)
            assert_same_tree(t, want)
            t.free()
    ctx.close()


@pytest.mark.parametrize("extra", [0, 4097])
def test_large_chunks(extra):
    torch_cuda()
    import paper_2512_23314_amd as bt
    n = (36 << 20) + extra
    T = np.resize(synth.random_text((5 << 20) + 13, 4, 3), n)
    T[n - 4096] ^= 1
    want = oracle.build_tree_par(T, 2, 4096).canonical
    ctx = bt.Context(0)
    tree = ctx.build(to_device(T), tau=2, leaf_len=4096)
    assert tree.serialize() == want
    tree.free()
    ctx.close()
