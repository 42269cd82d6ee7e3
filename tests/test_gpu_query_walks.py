"""rank, select and access at the edges of their walks: block lengths that are
and are not powers of two, leaves shorter and longer than the eight bytes counted
at a time, pointers that spill into the next block with one parent and with two,
absolute counters only, counters of every width, one tree and trees of a batch."""
import numpy as np
import pytest

import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


def _check(torch, tree, T):
    n = T.size
    rng = np.random.default_rng(n)
    pos = np.unique(np.concatenate([np.arange(min(n + 1, 700)), rng.integers(0, n + 1, 3000), [n]]))
    syms = np.unique(T)
    ch = syms[rng.integers(0, syms.size, pos.size)].astype(np.uint8)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    p64 = dev(pos.astype(np.int64)).to(torch.uint64)
    got = tree.rank(dev(ch), p64).to(torch.int64).cpu().numpy()
    total = {}
    for c in syms:
        at = np.flatnonzero(T == c)
        total[int(c)] = at
        assert np.array_equal(got[ch == c], np.searchsorted(at, pos[ch == c]))
    k = np.array([1 + rng.integers(0, total[int(c)].size) for c in ch])
    k[:syms.size] = [total[int(c)].size for c in ch[:syms.size]]
    got = tree.select(dev(ch), dev(k.astype(np.int64)).to(torch.uint64)).to(torch.int64).cpu().numpy()
    assert np.array_equal(got, [total[int(c)][x - 1] for c, x in zip(ch, k)])
    over = dev(np.array([total[int(c)].size + 1 for c in ch], np.int64)).to(torch.uint64)
    assert (tree.select(dev(ch), over).to(torch.int64).cpu().numpy() == -1).all()
    assert np.array_equal(tree.access(p64[:-1]).cpu().numpy(), T[pos[:-1]])


@pytest.mark.parametrize("tau,leaf", [(2, 1), (2, 7), (2, 8), (2, 9), (3, 5), (4, 16), (5, 23), (16, 32)])
def test_walks(tau, leaf):
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    ctx = bt.Context(0)
    texts = [synth.dna_copies(40011, 1777, 23, 2e-3, 1e-3, 9, tau * leaf),
             np.resize(synth.random_text(1013, 90, leaf), 20000 + leaf),
             synth.periodic_text(5003, 3, 1), synth.random_text(leaf + 1, 4, 3)]
    for T in texts:
        t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, rank_select=True)
        _check(torch, t, T)
        t.free()
    off = np.concatenate([[0], np.cumsum([T.size for T in texts])]).astype(np.uint64)
    for t, T in zip(ctx.build_batch(to_device(np.concatenate(texts)), off, tau=tau, leaf_len=leaf,
                                    rank_select=True), texts):
        _check(torch, t, T)
        t.free()
    # counters of 32 bits on the upper levels (b = 2^17 and more)
    if leaf == 16:
        T = synth.dna_copies(3 << 20, 300007, 11, 1e-4, 1e-5, 9, 5)
        t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, rank_select=True, s_hint=3)
        _check(torch, t, T)
        t.free()
    ctx.close()
