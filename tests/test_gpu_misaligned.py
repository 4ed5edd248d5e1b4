"""GPU parity where the output buffer starts 4 bytes past a 16-byte line: the
row scan then hands over an int32 field, and the column passes that stage with
vector loads give way to their forms for any alignment.  Bit-exact against the
oracle and equal to the aligned call; the kernel names show which form ran."""
import numpy as np
import pytest

from gpu_util import announce
from oracle import edt_oracle

pytestmark = pytest.mark.gpu


def call(metric, mask, offset):
    """(distances, kernel names) of an output `offset` elements into its allocation."""
    import torch

    from paper_2608_24738_amd import binding
    x = torch.from_numpy(mask).cuda()
    nd = mask.ndim - 1
    dtype = torch.float32 if metric == "euclidean" else torch.int32
    big = torch.zeros(mask.size + 8, dtype=dtype, device=x.device)
    out = big[offset:offset + mask.size].view(mask.shape)
    assert out.data_ptr() % 16 == 4 * offset
    binding.prof_enable(16)
    try:
        if metric == "euclidean":
            binding.tm_edt(x, nd, None, out, None)
        else:
            binding.tm_cdt(x, nd, binding.METRICS[metric], out)
        torch.cuda.synchronize()
        names = {n for n, _ in binding.prof_read()}
    finally:
        binding.prof_enable(0)
    assert not big[:offset].any() and not big[offset + mask.size:].any()
    return out.cpu().numpy(), names


CASES = [("euclidean", (16, 512, 512), "line_pair_final.i16", "line_pair_rag_final"),
         ("euclidean", (2, 64, 160, 192), "line_pair.i16", "line_pair_rag"),
         ("euclidean", (9, 900, 960), "line_bracket_final.i16", "line_bracket_final"),
         ("chessboard", (9, 900, 960), "cdt_bracket_final.i16", "cdt_bracket_final"),
         ("chessboard", (2, 300, 256), "cdt_line_final", "cdt_line_final"),
         ("taxicab", (4, 304, 256), "cdt_l1_scan_final.i16", "cdt_l1_scan_final"),
         ("taxicab", (2, 9, 304, 40), "cdt_l1_scan", "cdt_l1_scan")]


@pytest.mark.parametrize("metric,shape,aligned,misaligned", CASES,
                         ids=["%s-%s" % (c[0], "x".join(map(str, c[1]))) for c in CASES])
def test_misaligned_output(metric, shape, aligned, misaligned):
    rng = np.random.default_rng(sum(shape))
    mask = (rng.random(shape) >= 0.004).astype(np.uint8)
    mask[0] = 1                                           # without background
    mask[1, ..., : shape[-1] // 2] = 1                    # long distances
    announce("misaligned output %s %s" % (metric, shape))
    want, names = call(metric, mask, 0)
    assert aligned in names, names
    got, names = call(metric, mask, 1)
    assert misaligned in names, names
    assert not any(n.endswith("16") for n in names), names
    assert np.array_equal(got, want)
    if metric == "euclidean":
        assert np.array_equal(want, edt_oracle.edt(mask, len(shape) - 1, None, want_sq=False, nthreads=16)["dist"])
