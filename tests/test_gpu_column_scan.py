"""The dense scan's column walk (window lengths that are multiples of the tile,
texts of 2^25 windows or more) beside the tile-by-tile walk of other lengths:
segments cut by copies, ragged ends, with and without a short final key."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau,leaf,extra", [(4, 16, 0), (4, 16, 12345), (2, 64, 1024 + 7), (3, 10, 333)])
def test_columns(tau, leaf, extra):
    torch_cuda()
    import paper_2512_23314_amd as bt
    n = (9 << 22) + extra
    T = synth.dna_copies(n, n // 9, 9, 2e-4, 2e-5, 8, 97 + extra)
    # long exact copies, so that some blocks' windows are skipped at long lengths
    T[n // 2:n // 2 + 300000] = T[n // 5:n // 5 + 300000]
    want = oracle.build_tree_par(T, tau, leaf).canonical
    ctx = bt.Context(0)
    tree = ctx.build(to_device(T), sigma=4, tau=tau, leaf_len=leaf)
    assert tree.serialize() == want
    tree.free()
    ctx.close()
