"""select's search among a block's children, by quarters: arities on either side of
the powers of four, blocks with fewer children at the text's end, a symbol that all
children hold, one that few do; and its time at a large arity."""
import time

import numpy as np
import pytest

import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 33, 63, 64, 65, 255, 1000])
def test_every_occurrence(tau):
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    ctx = bt.Context(0)
    for leaf, n in ((1, 3 * tau + 1), (3, 7 * tau * 3 + 2), (8, min(2 * tau * tau * 8 + 5, 40000))):
        T = synth.random_text(n, 4, tau)
        T[T == 3] = 0
        T[np.random.default_rng(tau).integers(0, n, 1 + n // 500)] = 3
        t = ctx.build(to_device(T), tau=tau, leaf_len=leaf, rank_select=True)
        for c in np.unique(T):
            at = np.flatnonzero(T == c)
            k = torch.arange(1, at.size + 1, device="cuda").to(torch.uint64)
            got = t.select(torch.full((at.size,), int(c), dtype=torch.uint8, device="cuda"), k)
            assert np.array_equal(got.to(torch.int64).cpu().numpy(), at)
        t.free()
    ctx.close()


def test_time_at_a_large_arity():
    """select over rank, 2^18 queries on a text of 200 symbols at tau 64: 8.4 when a
    query read a marked block's counts four children after another, now 3.0.  The bound
    lies between."""
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    T = synth.random_text(16 << 20, 200, 7)
    ctx = bt.Context(0)
    t = ctx.build(to_device(T), tau=64, leaf_len=4, rank_select=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    m = 1 << 18
    pos = torch.randint(0, T.size, (m,), generator=g, device="cuda").to(torch.uint64)
    ch = torch.randint(0, 200, (m,), generator=g, device="cuda", dtype=torch.uint8)
    k = torch.randint(1, 80000, (m,), generator=g, device="cuda").to(torch.uint64)
    us = []
    for f in (lambda: t.rank(ch, pos), lambda: t.select(ch, k)):
        best = 1e9
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            best = min(best, 1e6 * (time.perf_counter() - t0))
        us.append(best)
    t.free()
    ctx.close()
    print("rank, select: %.1f %.1f us, ratio %.2f" % (us[0], us[1], us[1] / us[0]))
    assert us[1] < 5 * us[0]
