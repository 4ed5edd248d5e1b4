"""GPU parity of the packed line pass on lines of any length, stride and
alignment (k_line_pair16, one element per lane): line lengths around a patch of
16 rows, groups of 16 lines that cross blocks of rows, a partial last group,
distances past 255 (the exact re-search), and few site rows.  Bit-exact against
the oracle."""
import numpy as np
import pytest

from gpu_util import announce, check_against_oracle, run_gpu
from oracle import edt_oracle

pytestmark = pytest.mark.gpu

# (batch, spatial): at least 512 groups of 16 lines in every strided pass
CASES = [(2, (33, 40, 237)), (16, (17, 520)), (13, (511, 641)), (4, (31, 47, 95)), (40, (257, 207)), (1, (5, 160, 1650))]


@pytest.mark.parametrize("batch,spatial", CASES, ids=["%dx%s" % (b, "x".join(map(str, s))) for b, s in CASES])
def test_ragged_packed_lines(batch, spatial):
    from paper_2608_24738_amd import binding
    rng = np.random.default_rng(sum(spatial))
    mask = (rng.random((batch,) + spatial) >= 0.004).astype(np.uint8)
    mask[0] = 1
    mask[(0,) + tuple(n // 3 for n in spatial)] = 0            # one element: few site rows
    if batch > 2:
        mask[1] = 1                                            # no background
        mask[2] = 1
        mask[2, ..., : max(1, spatial[-1] // 8)] = 0           # far from a wide band
        mask[2, : (3 * spatial[0]) // 4] = 1
    nd = len(spatial)
    announce("ragged packed lines shape=%s" % (mask.shape,))
    binding.prof_enable(64)
    try:
        res = run_gpu(mask, nd, None, dist=True, idx=False, sq=True)
        names = {n for n, _ in binding.prof_read()}
    finally:
        binding.prof_enable(0)
    assert "line_pair_rag_final" in names, names
    assert nd == 2 or "line_pair_rag" in names, names
    check_against_oracle(mask, nd, None, res, edt_oracle.edt(mask, nd, None, nthreads=16))
