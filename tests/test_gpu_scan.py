"""GPU parity of the row scan of short ragged rows (k_scan_span): widths around
the 64-position chunk and the 1024-position span of a wave, waves whose lines
cross from one sample into the next (index carrier), rows without background,
and rank-1 inputs (all outputs from the scan).  Bit-exact against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, check_against_oracle, run_gpu
from oracle import edt_oracle

pytestmark = pytest.mark.gpu


def random_mask(shape, seed):
    rng = np.random.default_rng(seed)
    m = (rng.random(shape) >= 0.06).astype(np.uint8)
    m.reshape(-1, shape[-1])[::3] = 1          # every third row without background
    return m


@pytest.mark.parametrize("n", [1, 2, 3, 31, 63, 65, 129, 511, 1000, 1023])
def test_widths(n):
    mask = random_mask((3, 70, n), n)
    mask[1] = 1                                 # a sample without background
    announce("scan rows of %d" % n)
    ora = edt_oracle.edt(mask, 2, None, nthreads=16)
    check_against_oracle(mask, 2, None, run_gpu(mask, 2, None, dist=True, idx=True, sq=True), ora)
    check_against_oracle(mask, 2, None, run_gpu(mask, 2, None, dist=True, idx=False), ora)
    line = random_mask((37, n), n + 1)
    announce("scan rank 1, %d" % n)
    check_against_oracle(line, 1, None, run_gpu(line, 1, None, dist=True, idx=True, sq=True),
                         edt_oracle.edt(line, 1, None, nthreads=16))


def test_many_samples_per_wave():
    # 5 lines of 7 elements per sample: every wave spans several samples
    mask = random_mask((1200, 5, 7), 9)
    announce("scan 1200 x 5 x 7 x 1 plane")
    mask3 = mask.reshape(1200, 5, 1, 7)
    check_against_oracle(mask3, 3, None, run_gpu(mask3, 3, None, dist=True, idx=True),
                         edt_oracle.edt(mask3, 3, None, nthreads=16))
