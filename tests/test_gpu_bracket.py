"""GPU parity of the bracketed column search (k_line_bracket): long lines of the
first strided pass, and the index pass of 2-D inputs with more than 256 rows.
Masks put every phase to work: near patches only (dense), far ones (a few discs),
few site rows (one pixel), no background, one background block in a corner (the
longest brackets), all background, a band without background a quarter of the
lines long (few far patches, searched on; 2048 rows: past 249 rows, so left to the
brackets after all).  Bit-exact against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, check_against_oracle, run_gpu
from oracle import edt_oracle

pytestmark = pytest.mark.gpu


def masks(spatial, seed):
    rng = np.random.default_rng(seed)
    grid = np.ogrid[tuple(slice(0, n) for n in spatial)]
    out = [rng.random(spatial) >= 0.3, rng.random(spatial) >= 0.004]
    far = np.ones(spatial, bool)
    for _ in range(6):
        c = [rng.uniform(0, n) for n in spatial]
        r = rng.uniform(0.02, 0.12) * min(spatial) + 1
        far &= ~(sum((g - x) ** 2 for g, x in zip(grid, c)) <= r * r)
    one = np.ones(spatial, bool)
    one[tuple(rng.integers(0, n) for n in spatial)] = False
    corner = np.ones(spatial, bool)
    corner[tuple(slice(0, min(40, n)) for n in spatial)] = False
    band = out[0].copy()
    band[..., spatial[-2] // 3 : spatial[-2] // 3 + spatial[-2] // 4 - 8, :] = True
    out += [far, one, np.ones(spatial, bool), corner, np.zeros(spatial, bool), band]
    return np.stack(out).astype(np.uint8)


def names_of(fn):
    from paper_2608_24738_amd import binding
    binding.prof_enable(64)
    try:
        res = fn()
        return res, {n for n, _ in binding.prof_read()}
    finally:
        binding.prof_enable(0)


# rows at the rule's edges (640, and 896 for rows of a multiple of 64, which go over
# packed where a scan wave's rows pair up), one segment short and over, partial last
# groups, the longest line; the middle axis of 3-D inputs
SHAPES = [((640, 513), ""), ((647, 515), ""), ((897, 576), ""), ((1024, 512), ".16"), ((2048, 517), ""),
          ((3, 645, 521), ""), ((2, 900, 512), ".16")]


def chessboard(mask):
    """(B, *spatial) chessboard distances, axis by axis, by shifts on the GPU."""
    import torch
    f = torch.where(torch.from_numpy(mask).cuda() == 0, 0, 1 << 20).to(torch.int32)
    for axis in range(1, f.dim()):
        best, n = f.clone(), f.shape[axis]
        for k in range(1, n):
            lo, hi = f.narrow(axis, 0, n - k), f.narrow(axis, k, n - k)
            to_lo, to_hi = best.narrow(axis, 0, n - k), best.narrow(axis, k, n - k)
            torch.minimum(to_hi, lo.clamp(min=k), out=to_hi)
            torch.minimum(to_lo, hi.clamp(min=k), out=to_lo)
        f = best
    return torch.where(f < (1 << 20), f, -1).cpu().numpy()


@pytest.mark.parametrize("spatial,packed", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_distances(spatial, packed):
    import torch

    from paper_2608_24738_amd import binding
    nd = len(spatial)
    once = masks(spatial, sum(spatial))
    # the rule also asks for 512 groups of 16 lines: the masks several times over
    reps = -(-512 * 16 * spatial[-2] // once.size) + 1
    mask = np.tile(once, (reps,) + (1,) * nd)
    announce("bracket distances shape=%s" % (mask.shape,))
    kernel = "bracket" + ("_final" if nd == 2 else "") + packed.replace(".", ".i")
    res, names = names_of(lambda: run_gpu(mask, nd, None, dist=True, idx=False, sq=True))
    assert "line_" + kernel in names, names
    assert ("scan_word.o16" in names) == bool(packed), names
    ora = edt_oracle.edt(once, nd, None, nthreads=16)
    ora = {k: np.tile(ora[k], (reps,) + (1,) * nd) for k in ("dist", "sq")}
    check_against_oracle(mask, nd, None, res, ora)
    x = torch.from_numpy(mask).cuda()
    out = torch.empty(mask.shape, dtype=torch.int32, device=x.device)
    _, names = names_of(lambda: (binding.tm_cdt(x, nd, 2, out), torch.cuda.synchronize()))
    assert "cdt_" + kernel in names, names
    want = np.tile(chessboard(once), (reps,) + (1,) * nd)
    assert np.array_equal(out.cpu().numpy(), want)


# value and row in one key, and too large for one (11 bits of row beside 22 of value)
@pytest.mark.parametrize("spatial", [(257, 48), (300, 33), (375, 500), (1024, 100), (1100, 1090), (2048, 40)],
                         ids=lambda s: "%dx%d" % s)
def test_indices(spatial):
    mask = masks(spatial, sum(spatial) + 1)
    announce("bracket indices shape=%s" % (mask.shape,))
    res, names = names_of(lambda: run_gpu(mask, 2, None, dist=True, idx=True))
    assert "line_bracket_idx_final" in names, names
    check_against_oracle(mask, 2, None, res, edt_oracle.edt(mask, 2, None, nthreads=16))
    only, _ = names_of(lambda: run_gpu(mask, 2, None, dist=False, idx=True))
    assert np.array_equal(only["idx"], res["idx"])


def test_widest_rows():
    """Rows of 16000, lines of 2048 (the rule's largest): one background block of 40
    x 40 in a corner, so that values reach the largest a key and a 16-bit distance
    hold.  Its nearest element is known in closed form."""
    import torch

    from paper_2608_24738_amd import binding
    n, w = 2048, 16000
    dev = torch.device("cuda:0")
    x = torch.ones((1, n, w), dtype=torch.uint8, device=dev)
    x[0, :40, :40] = 0
    r, c = torch.arange(n, device=dev)[:, None], torch.arange(w, device=dev)[None]
    dr, dc = (r - 39).clamp(min=0), (c - 39).clamp(min=0)
    sq = (dr * dr + dc * dc).to(torch.int32)
    announce("bracket widest rows 1x%dx%d" % (n, w))
    out = torch.empty((1, n, w), dtype=torch.int32, device=dev)
    _, names = names_of(lambda: (binding.tm_edt_sq(x, 2, out), torch.cuda.synchronize()))
    assert "line_bracket_final" in names, names
    assert torch.equal(out[0], sq)
    _, names = names_of(lambda: (binding.tm_cdt(x, 2, 2, out), torch.cuda.synchronize()))
    assert "cdt_bracket_final" in names, names
    assert torch.equal(out[0], torch.maximum(dr, dc).to(torch.int32))
    dist = torch.empty((1, n, w), dtype=torch.float32, device=dev)
    idx = torch.empty((1, 2, n, w), dtype=torch.int32, device=dev)
    _, names = names_of(lambda: (binding.tm_edt(x, 2, None, dist, idx), torch.cuda.synchronize()))
    assert "line_bracket_idx_final" in names, names
    assert torch.equal(dist[0], sq.double().sqrt().float())
    assert torch.equal(idx[0, 0], r.clamp(max=39).expand(n, w).to(torch.int32))
    assert torch.equal(idx[0, 1], c.clamp(max=39).expand(n, w).to(torch.int32))
