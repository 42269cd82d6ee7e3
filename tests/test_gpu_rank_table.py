"""The sampled count table behind rank/select at the edges of its rows (1024
bytes) and row blocks (64 rows): every symbol's rank at the rows' ends, for texts
that end inside, at and one past a row and a block of rows, and for one symbol."""
import numpy as np
import pytest

import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu
ROW, BLOCK = 1024, 64 * 1024


@pytest.mark.parametrize("n", [1, ROW - 1, ROW, ROW + 1, BLOCK - 1, BLOCK, BLOCK + 1, 65 * BLOCK, 65 * BLOCK + 17])
@pytest.mark.parametrize("sigma", [1, 65, 256])
def test_rank_at_rows(n, sigma):
    torch = torch_cuda()
    import paper_2512_23314_amd as bt
    T = synth.random_text(n, sigma, n + sigma) if sigma > 1 else np.full(n, 200, np.uint8)
    ctx = bt.Context(0)
    t = ctx.build(to_device(T), sigma=256, tau=4, leaf_len=16, rank_select=True, s_hint=7)
    pos = np.unique(np.clip(np.arange(0, n + ROW, ROW // 2)[:, None] + np.array([-1, 0, 1, 17]), 0, n))
    syms = np.unique(T)[:: max(1, sigma // 16)]
    ch = np.repeat(syms, pos.size).astype(np.uint8)
    pp = np.tile(pos, syms.size)
    got = t.rank(torch.from_numpy(ch).cuda(), torch.from_numpy(pp.astype(np.int64)).cuda().to(torch.uint64))
    want = np.concatenate([np.searchsorted(np.flatnonzero(T == c), pos) for c in syms])
    assert np.array_equal(got.to(torch.int64).cpu().numpy(), want)
    t.free()
    ctx.close()
