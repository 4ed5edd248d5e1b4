"""GPU parity of the brute-force transform's key form (exact euclidean, ranks 2
and 3): more background elements than one run of 1024, chunks of 4096 bytes with
a ragged end and unaligned samples, ties, the largest extents a key holds and the
first ones past it.  Bit-exact with canonical indices against the oracle."""
import numpy as np
import pytest

from gpu_util import announce
from oracle import edt_oracle

pytestmark = pytest.mark.gpu

CASES = [(2, (67, 97), 0.5), (3, (41, 101), 0.9), (2, (19, 21, 23), 0.3), (1, (4, 1447), 0.2), (1, (3, 1449), 0.2),
         (2, (7, 9, 11), 1.0), (3, (1, 5), 0.4)]


@pytest.mark.parametrize("batch,spatial,p_bg", CASES, ids=["%dx%s" % (b, "x".join(map(str, s))) for b, s, _ in CASES])
def test_keys(batch, spatial, p_bg):
    import torch

    from paper_2608_24738_amd import binding
    rng = np.random.default_rng(sum(spatial))
    mask = (rng.random((batch,) + spatial) >= p_bg).astype(np.uint8)
    mask[-1] = 1                                       # without background
    if batch > 1:
        mask[-1, ..., -1] = 0                          # many ties
    announce("bf keys shape=%s" % (mask.shape,))
    x = torch.from_numpy(mask[:, None].copy()).cuda()
    d, i = binding.distance_transform_bf(x, "euclidean", return_indices=True)
    ora = edt_oracle.dt_bf(mask, len(spatial), "euclidean", None)
    assert np.array_equal(d.cpu().numpy()[:, 0], ora["dist"])
    assert np.array_equal(i.cpu().numpy()[:, 0], ora["idx"])
