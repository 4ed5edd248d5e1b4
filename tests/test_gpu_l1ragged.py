"""GPU parity of the taxicab whole-line pass on lines of any stride (groups of 8
lines that are no multiple of the row, cross samples, or end past the last
line), at the edges of the rows a lane holds (4, 8, 12, 16, 36 x 64), final and
not; lines of fewer than 40 rows take the windowed search.  Bit-exact against the
oracle."""
import numpy as np
import pytest

from gpu_util import announce
from oracle import edt_oracle

pytestmark = pytest.mark.gpu

SCAN, WINDOWED = "cdt_l1_scan", "cdt_line"
# (spatial, kernel of each strided pass, the last axis but one first)
SHAPES = [((256, 7), [SCAN]), ((257, 33), [SCAN]), ((512, 9), [SCAN]), ((513, 129), [SCAN]), ((768, 1), [SCAN]),
          ((769, 5), [SCAN]), ((1024, 17), [SCAN]), ((1025, 3), [SCAN]), ((2304, 6), [SCAN]), ((40, 31), [SCAN]),
          ((39, 31), [WINDOWED]), ((17, 31), [WINDOWED]), ((5, 300, 7), [SCAN, WINDOWED]), ((41, 300, 7), [SCAN, SCAN])]


@pytest.mark.parametrize("spatial,passes", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_ragged_taxicab(spatial, passes):
    import torch

    from paper_2608_24738_amd import binding
    rng = np.random.default_rng(sum(spatial))
    mask = (rng.random((3,) + spatial) >= 0.01).astype(np.uint8)
    mask[1] = 1                                   # a sample without background
    mask[(2,) + tuple(n - 1 for n in spatial)] = 0
    announce("ragged taxicab shape=%s" % (mask.shape,))
    x = torch.from_numpy(mask).cuda()
    out = torch.empty(mask.shape, dtype=torch.int32, device=x.device)
    binding.prof_enable(16)
    try:
        binding.tm_cdt(x, len(spatial), 1, out)
        torch.cuda.synchronize()
        names = [n for n, _ in binding.prof_read()]
    finally:
        binding.prof_enable(0)
    assert names[1:] == passes[:-1] + [passes[-1] + "_final"], names
    assert np.array_equal(out.cpu().numpy(), edt_oracle.cdt(mask, len(spatial), "taxicab", nthreads=16))
