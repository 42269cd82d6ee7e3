"""Device memory of a build, the most in use at once."""
import pytest

import synth
from tests.gpu_util import to_device, torch_cuda

pytestmark = pytest.mark.gpu


def test_peak_of_pruning():
    """A pruned build keeps every level until its end.  32 MiB of random DNA, whose
    levels are full: 550 MB; 581 with what the leaf level would be scanned by kept too."""
    torch_cuda()
    import paper_2512_23314_amd as bt
    T = synth.random_text((32 << 20) - 5, 4, 14)
    ctx = bt.Context(0)
    ctx.build(to_device(T), tau=4, leaf_len=8, prune=True).free()
    peak = ctx.memory()["peak"]
    ctx.close()
    print("peak of a pruned build: %.1f MB" % (peak / 1e6))
    assert peak <= 565e6
