"""Scans in rounds on a repetitive text whose levels have enough keys and windows for
them (2^19 and 2^28) in both phases, against the threaded oracle: most keys occur in
the first copies, and the filters of later rounds drop them."""
import pytest

import oracle
import synth
from tests.gpu_util import assert_same_tree, to_device, torch_cuda

pytestmark = pytest.mark.gpu


def test_copies_of_every_age():
    torch_cuda()
    import paper_2512_23314_amd as bt
    tau, leaf = 2, 64
    T = synth.dna_copies(5 << 26, 1 << 23, 40, 1e-3, 1e-4, 8, 5)
    want = oracle.build_tree_par(T, tau, leaf)
    # a level's runs are at most the unmarked blocks above it and one more; phase 2
    # has a key for every block where a quarter is unmarked, unless the level is the
    # last one scanned
    lv = want.levels
    keys = {1: [], 2: []}
    for up, L in zip(lv[:-2], lv[1:-1]):
        if L.c * L.b >= 1 << 28:
            keys[1].append(L.c - up.u - 1)
            keys[2].append(L.c if 4 * L.u >= L.c and L is not lv[-2] else L.u)
    assert sum(k >= 1 << 19 for k in keys[1]) >= 2 and max(keys[2]) >= 1 << 19
    ctx = bt.Context(0)
    d = to_device(T)
    for lean in (False, True):
        t = ctx.build(d, sigma=4, tau=tau, leaf_len=leaf, lean=lean)
        assert_same_tree(t, want)
        t.free()
    ctx.close()
