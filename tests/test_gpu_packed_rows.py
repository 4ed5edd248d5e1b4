"""GPU parity where the row scan's waves hold an odd number of rows (row widths
of 384, 576 and 640: five and three rows per wave) and the extent of the next
axis is a multiple of it: the packed row field pairs rows 2R and 2R + 1, which
such waves cannot do, so the field has to go over unpacked.  Widths of 448, 704
and 768 leave lanes of a wave without a row (14, 22 and 24 words do not divide
64); they must not write past the wave's rows."""
import numpy as np
import pytest

from gpu_util import announce
from oracle import edt_oracle

pytestmark = pytest.mark.gpu

CASES = [((130, 384), 2), ((66, 576), 3), ((129, 640), 6), ((384, 448), 2), ((64, 768), 3), ((520, 704), 2)]


@pytest.mark.parametrize("metric", ["euclidean", "taxicab", "chessboard"])
@pytest.mark.parametrize("spatial,batch", CASES, ids=["%dx%d" % s for s, _ in CASES])
def test_odd_rows_per_wave(spatial, batch, metric):
    import torch

    from paper_2608_24738_amd import binding
    rng = np.random.default_rng(spatial[1])
    mask = (rng.random((batch,) + spatial) >= 0.003).astype(np.uint8)
    x = torch.from_numpy(mask[:, None].copy()).cuda()
    announce("odd rows per wave %s shape=%s" % (metric, mask.shape))
    if metric == "euclidean":
        got = binding.distance_transform_edt(x).cpu().numpy()[:, 0]
        want = edt_oracle.edt(mask, 2, None, nthreads=16)["dist"]
    else:
        got = binding.distance_transform_cdt(x, metric).cpu().numpy()[:, 0]
        want = edt_oracle.cdt(mask, 2, metric, nthreads=16)
    assert np.array_equal(got, want)
