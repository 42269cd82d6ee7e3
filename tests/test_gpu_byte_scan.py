"""The byte scan's chunks of 2048 windows, 32 per lane: texts that end around them,
at every alignment, with few candidates, with runs of candidates (every window of a
lane) and with segments that end inside a lane."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["dna", "runs", "copies"])
@pytest.mark.parametrize("n", [2048, 2048 + 64 + 31, 4096 + 33, 3 * 2048 - 1, 20 * 2048 + 17])
def test_chunks(kind, n):
    torch_cuda()
    import paper_2512_23314_amd as bt
    rng = np.random.default_rng(n)
    if kind == "dna":
        T = synth.random_text(n, 4, 5)
    elif kind == "runs":  # long runs: all of a lane's windows pass
        T = np.repeat(rng.integers(0, 3, n // 40 + 1, dtype=np.uint8), 40)[:n].copy()
    else:  # copies of the first part: windows that are skipped cut the segments
        T = np.resize(synth.random_text(n // 5 + 3, 4, 9), n)
        T[rng.integers(0, n, 9)] ^= 1
    ctx = bt.Context(0)
    for off in range(4):
        d = to_device(np.concatenate([np.zeros(off, np.uint8), T]))
        for tau, leaf in ((2, 16), (4, 20)):
            want = oracle.build_tree(T, tau, leaf).canonical
            tree = ctx.build(d[off:], tau=tau, leaf_len=leaf)
            assert tree.serialize() == want
            tree.free()
    ctx.close()
