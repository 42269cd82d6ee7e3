"""The short final key of a text (the key that ends in the text's short last
block), which the scans test by its first bytes before the whole key: tails
around the lengths where that test changes, with copies of the tail earlier in
the text and near-copies that agree in the tested bytes only."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import assert_same_tree, to_device, torch_cuda

pytestmark = pytest.mark.gpu
TAILS = [1, 7, 8, 9, 31, 63, 64, 65, 66, 200]


def _text(n, tail, seed):
    """n bytes whose last `tail` bytes occur before, and whose last block's
    first bytes also occur followed by something else."""
    T = synth.random_text(n, 4, seed)
    for at in (n // 7, n // 3):  # copies of the end, some longer than any key
        T[at:at + tail + 700] = T[n - tail - 700:n]
    near = T[n - tail - 700:n].copy()
    near[-max(1, tail // 8):] = T[:max(1, tail // 8)][::-1]
    T[n // 11:n // 11 + near.size] = near
    return T


@pytest.mark.parametrize("tail", TAILS)
@pytest.mark.parametrize("tau,leaf", [(2, 16), (4, 64)])
def test_tails(tail, tau, leaf):
    torch_cuda()
    import paper_2512_23314_amd as bt
    b = leaf * tau ** 3
    texts = [_text(40 * b + tail, tail, 17 * tail + tau), _text(23 * b + tail, tail, 31 * tail + tau),
             np.resize(np.frombuffer(b"ab" * 33 + b"a", np.uint8), 19 * b + tail)]
    want = [oracle.build_tree(T, tau, leaf) for T in texts]
    ctx = bt.Context(0)
    for lean in (False, True):
        for T, w in zip(texts, want):
            t = ctx.build(to_device(T), sigma=256, tau=tau, leaf_len=leaf, lean=lean)
            assert_same_tree(t, w)
            t.free()
        off = np.concatenate([[0], np.cumsum([T.size for T in texts])]).astype(np.uint64)
        for t, w in zip(ctx.build_batch(to_device(np.concatenate(texts)), off, sigma=256, tau=tau,
                                        leaf_len=leaf, lean=lean), want):
            assert_same_tree(t, w)
            t.free()
    ctx.close()
