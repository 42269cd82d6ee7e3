"""Scans in rounds (2^28 windows and 2^19 keys or more of one text) against the
scan without queues, which takes every window in one pass: repetitive text with
copies of every age, a text whose keys hardly repeat, and the lean build."""
import numpy as np
import pytest

import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _sparse(n, seed):
    T = synth.random_text(n, 4, seed)
    for k in range(1, 40):  # some copies, the last ones near the end
        a, b = n * k // 41, (n * k * 7 // 41 + n // 83) % (n - 100000)
        T[a:a + 90000] = T[b:b + 90000]
    return T


@pytest.mark.parametrize("kind,tau,leaf", [("copies", 2, 16), ("sparse", 4, 32)])
def test_rounds(kind, tau, leaf):
    torch_cuda()
    import paper_2512_23314_amd as bt
    n = (1 << 28) + (5 << 20) + 321
    T = synth.dna_copies(n, 1 << 23, 33, 1e-3, 1e-4, 8, 5) if kind == "copies" else _sparse(n, 6)
    ctx = bt.Context(0)
    d = to_device(T)
    want = None
    for kw in ({"debug_flags": bt.BT_DBG_NO_QUEUE}, {}, {"lean": True}):
        t = ctx.build(d, sigma=4, tau=tau, leaf_len=leaf, **kw)
        got = t.serialize()
        t.free()
        want = want or got
        assert got == want
    ctx.close()
