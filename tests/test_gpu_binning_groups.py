"""The binning on grids of more tile rows (or pieces of rows) than one group of
strips holds, for few and for many Gaussians, and with more rows per Gaussian
than the count keeps: lists, ranges, keys, flags and depth prefixes against the
oracle, and the lists of a resumed call."""
import pytest
import torch

import synth
import test_gpu_binning as base
from test_gpu_binning import B  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

FEW = 1 << 17   # up to this many Gaussians take groups of 4096 strips and keep 36 rows each, more 1024 and 24
# name: Gaussians, image width and height, mean log-scale, share of the tiles
CASES = {
    "few_4096_rows": (400, 24, 65536, -3.0, None),
    "few_4097_rows": (400, 24, 65537, -3.0, 0.5),
    "few_4098_pieces": (300, 4112, 2049 * 16, -4.0, None),
    "few_long": (300, 64, 4096, -2.3, None),
    "few_long_subset": (300, 64, 4096, -2.0, 0.3),
    "few_last": (FEW, 24, 16400, -6.5, None),
    "many_1024_rows": (FEW + 1, 24, 16384, -6.5, 0.6),
    "many_1025_rows": (FEW + 1, 24, 16400, -6.5, None),
    "many_1026_pieces": (FEW + 1, 4112, 513 * 16, -8.0, 0.4),
    "many_long": (FEW + 1, 24, 4096, -3.2, None),
    "sub_257_rows": (700, 40, 4097, -1.5, None),
}


@pytest.mark.parametrize("case", list(CASES))
def test_lists_of_grouped_strips(B, case, monkeypatch):  # noqa: F811
    monkeypatch.setitem(base.CASES, case, CASES[case])
    base.test_lists_at_route_boundaries(B, case)


@pytest.mark.parametrize("case", list(CASES))
def test_resumed_lists_of_grouped_strips(B, case):  # noqa: F811
    from paper_2606_15924_amd.pipeline import ViewBuffers
    n, W, H, scale, _ = CASES[case]
    side = max(W, H)
    cam = B.camera(synth.look_at((2.6, 0.4, 0.9), fx=1.1 * side, fy=1.1 * side, width=W, height=H))
    rp = B.raster_params()
    vb = ViewBuffers(n, W, H, 1, -1, "cuda", capacity=1 << 22)
    vb.project(base.dev(synth.gaussians(n, 11, logscale_mean=scale)), cam, rp)
    vb.bin_sort_async(None, rp.alpha_min)
    m = vb.n_pairs
    want, ranges = vb.vals[:m].clone(), vb.ranges.clone()
    assert m > 50
    vb._alloc_pairs(m // 3)
    vb.ranges.fill_(-1)
    vb.bin_sort(None, rp.alpha_min)   # does not fit: resumed
    assert vb.n_pairs == m and torch.equal(vb.vals[:m], want) and torch.equal(vb.ranges, ranges)
