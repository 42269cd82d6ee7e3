"""Verification of keys around the lengths where its lane groups change (64, 128,
256, 512, 1024 bytes), where it goes from one launch to the list (4096), and of
short final keys in between: every key of these texts occurs earlier, at any
alignment, and with 12-bit fingerprints most verifications fail first."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_same_tree, to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf,tau", [(2, 2), (16, 2), (31, 2), (33, 2), (65, 2), (129, 3), (257, 2), (1000, 2),
                                      (1025, 2), (2048, 2)])
def test_key_lengths(leaf, tau):
    torch_cuda()
    import paper_2512_23314_amd as bt
    ctx = bt.Context(0)
    b = leaf * tau
    for n, sub in ((70 * b + leaf // 2 + 1, 0), (70 * b, 1), (131 * b + 3, 1)):
        w = synth.random_text(5 * b + 7, 4, leaf)
        T = np.resize(w, n)
        if sub:  # a few changed bytes, so that some keys are new
            T[np.arange(3 * b, n, 11 * b + 5)] ^= 1
        want = oracle.build_tree(T, tau, leaf)
        for flags in (0, bt.BT_DBG_WEAK_HASH):
            t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, debug_flags=flags)
            assert_same_tree(t, want)
            t.free()
    ctx.close()
