"""Builds whose prefix fingerprints end around a 4 KiB row of a wave and a 32 KiB
tile: the single build stores every 4th value through LDS.  Copies up to the very end
of the text make the last values decide the tree; an offset view takes the byte loads."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 3])
@pytest.mark.parametrize("n", [4096 - 1, 4096, 4096 + 33, 32768 - 64, 32768 - 1, 32768, 32768 + 1,
                               32768 + 4, 65536 + 4096 + 31, 5 * 32768 + 64])
def test_ends(n, off):
    torch_cuda()
    import paper_2512_23314_amd as bt
    rng = np.random.default_rng(n)
    T = rng.integers(0, 4, n, dtype=np.uint8)
    T[n - n // 3:] = T[:n // 3]
    buf = np.concatenate([np.zeros(off, np.uint8), T])
    ctx = bt.Context(0)
    d = to_device(buf)
    for tau, leaf in ((2, 3), (4, 16)):
        tree = ctx.build(d[off:], sigma=4, tau=tau, leaf_len=leaf)
        assert tree.serialize() == oracle.build_tree(T, tau, leaf).canonical
        tree.free()
    ctx.close()
