"""The byte scan where many windows pass its filter: texts of runs, whose windows
repeat a key's first eight bytes.  Chunks take their candidates in the order of the
samples from 16 lanes with many on; chunks on either side of that, chunks that mix such
lanes with others and with lanes that cross segments, texts of a batch."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _sparse(n, every, seed):
    rng = np.random.default_rng(seed)
    T = np.zeros(n, np.uint8)
    T[rng.integers(0, n, max(1, n // every))] = rng.integers(1, 4, max(1, n // every))
    return T


def _lanes(n, lanes, seed):
    """Runs of `lanes` times 32 bytes in each 2048, the rest random; zeros at the end."""
    T = synth.random_text(n, 250, seed)
    at = np.arange(n) % 2048
    T[(at >= 100) & (at < 100 + 32 * lanes)] = 0
    T[-40:] = 0
    return T


@pytest.mark.parametrize("lean", [False, True])
@pytest.mark.parametrize("kind", ["sparse20", "sparse300", "lanes15", "lanes17", "lanes60"])
def test_dense_candidates(kind, lean):
    torch_cuda()
    import paper_2512_23314_amd as bt
    ctx = bt.Context(0)
    make = (lambda n, s: _sparse(n, int(kind[6:]), s)) if kind[0] == "s" else (lambda n, s: _lanes(n, int(kind[5:]), s))
    texts = [make(n, n) for n in (40 * 2048, 9 * 2048 + 33, 100001, 3 * 2048 - 31)]
    for T in texts:
        for tau, leaf in ((2, 16), (4, 20)):
            t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, lean=lean)
            assert t.serialize() == oracle.build_tree(T, tau, leaf).canonical
            t.free()
    off = np.concatenate([[0], np.cumsum([T.size for T in texts])]).astype(np.uint64)
    trees = ctx.build_batch(to_device(np.concatenate(texts)), off, tau=2, leaf_len=16, lean=lean)
    for T, t in zip(texts, trees):
        assert t.serialize() == oracle.build_tree(T, 2, 16).canonical
    bt.free_trees(trees)
    ctx.close()


def test_time_of_dense_candidates():
    """The scan's time over the prefix scan's on a text that is zero but for every
    256th byte: 32 at 64 MiB; with one window of each lane in a step, 32 bytes apart,
    it was 69.  The bound lies between."""
    torch_cuda()
    import paper_2512_23314_amd as bt
    T = _sparse((64 << 20) + 12345, 256, 1)
    ctx = bt.Context(0)
    d = to_device(T)
    ratios = []
    for _ in range(5):
        ctx.profile(True)
        ctx.reset_stats()
        ctx.build(d, tau=2, leaf_len=8).free()
        ratios.append(ctx.kernel_stats("byte_scan")["ms"] / ctx.kernel_stats("prefix_fp")["ms"])
    ctx.close()
    print("byte scan / prefix scan:", ["%.1f" % r for r in ratios])
    assert sorted(ratios)[2] < 48
