"""The binning's routes at the sizes where each begins or ends: the depth
order by counted ranks or by radix passes, blocks of depth positions and of
row records, row intervals kept or evaluated again, the id buffer of a block
of records, grids of more than 256 tile columns or rows, tile subsets and
depth prefixes.  Lists, ranges, keys and touched flags against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import project
from oracle.params import RasterParams
from support import check_pair_lists, splat_record

pytestmark = pytest.mark.gpu

RP = RasterParams()

# name: Gaussians, image width and height, mean log-scale, share of the tiles
CASES = {
    "one": (1, 48, 48, -2.0, None),
    "block_255": (255, 64, 64, -3.0, None),
    "block_256": (256, 64, 64, -3.0, None),
    "block_257": (257, 64, 64, -3.0, 0.4),
    "ranks_16384": (16384, 64, 48, -5.0, None),
    "passes_16385": (16385, 64, 48, -5.0, 0.5),
    "columns_128": (1500, 2048, 96, -2.5, None),
    "columns_129": (1500, 2049, 96, -2.5, 0.3),
    "columns_256": (700, 4096, 40, -2.5, 0.6),
    "columns_257": (700, 4097, 40, -2.5, None),
    "columns_600": (500, 9600, 40, -2.0, 0.5),
    "rows_256": (700, 40, 4096, -2.5, None),
    "rows_257": (700, 40, 4097, -2.5, 0.5),
    "rows_600": (500, 40, 9600, -2.0, None),
    "large_splats": (3000, 640, 512, -1.2, None),
    "large_splats_subset": (3000, 640, 512, -1.2, 0.05),
}


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("case", list(CASES))
def test_lists_at_route_boundaries(B, case):
    n, W, H, scale, share = CASES[case]
    p = synth.gaussians(n, 11, logscale_mean=scale)
    side = max(W, H)
    cam = synth.look_at((2.6, 0.4, 0.9), fx=1.1 * side, fy=1.1 * side, width=W, height=H)
    pr = project.project(p, cam, RP)
    TX, TY = pr["TX"], pr["TY"]
    valid = tile_slot = None
    if share is not None:
        rng = np.random.default_rng(4)
        valid = np.sort(rng.choice(TX * TY, max(1, int(share * TX * TY)), replace=False))
        slots = -np.ones(TX * TY, dtype=np.int32)
        slots[valid] = np.arange(valid.size)
        tile_slot = dev(slots)
    rect, splat, depth = dev(pr["rect"].T.astype(np.int32)), dev(splat_record(pr)), dev(pr["depth32"])
    area = (pr["rect"][2] - pr["rect"][0]) * (pr["rect"][3] - pr["rect"][1])
    cap = int(area[pr["visible"]].sum()) + 3
    ws = torch.empty(B.tgs_bin_sort_workspace_size(n, cap, TX * TY), dtype=torch.uint8, device="cuda")
    keys = torch.empty(cap, dtype=torch.int64, device="cuda")
    vals = torch.empty(cap, dtype=torch.int32, device="cuda")
    ranges = torch.full((TX * TY, 2), -1, dtype=torch.int32, device="cuda")
    touched = torch.zeros(n, dtype=torch.uint8, device="cuda")
    n_pairs = B.tgs_bin_sort(rect, splat, depth, n, tile_slot, TX, TY, 1.0 / 255.0, keys, vals, cap, ranges, touched,
                             ws)
    v, r = host(vals).copy(), host(ranges).copy()
    check_pair_lists(v, r, n_pairs, pr, valid, keys=host(keys), max_dropped_checked=4000)
    flags = np.zeros(n, dtype=np.uint8)
    flags[v[:n_pairs]] = 1
    assert np.array_equal(host(touched), flags)

    # a capacity one too small: empty ranges, the count still reported
    if n_pairs > 0:
        ws1 = torch.empty(B.tgs_bin_sort_workspace_size(n, n_pairs - 1, TX * TY), dtype=torch.uint8, device="cuda")
        counts = torch.zeros(2, dtype=torch.int64, device="cuda")
        B.tgs_bin_sort_async(rect, splat, depth, n, tile_slot, TX, TY, 1.0 / 255.0, None, vals, n_pairs - 1, ranges,
                             None, counts, ws1)
        assert host(ranges).max() == 0 and host(counts).tolist() == [n_pairs, n_pairs]
        assert np.array_equal(host(vals), v)

    # a depth prefix and the continuation of every listed tile: together the whole lists
    m = max(1, n // 3)
    counts = torch.zeros(3, dtype=torch.int64, device="cuda")
    B.tgs_bin_sort_prefix_async(rect, splat, depth, n, tile_slot, TX, TY, 1.0 / 255.0, m, None, vals, cap, ranges,
                                None, counts, ws)
    flags_t = tile_slot if tile_slot is not None else torch.zeros(TX * TY, dtype=torch.int32, device="cuda")
    ws2 = torch.empty(B.tgs_bin_sort_workspace_size(n, cap, TX * TY), dtype=torch.uint8, device="cuda")
    vals2 = torch.empty(cap, dtype=torch.int32, device="cuda")
    ranges2 = torch.full((TX * TY, 2), -1, dtype=torch.int32, device="cuda")
    counts2 = torch.zeros(2, dtype=torch.int64, device="cuda")
    B.tgs_bin_sort_continue_async(splat, n, flags_t, TX, TY, 1.0 / 255.0, m, cap, ws, vals2, cap, ranges2, counts2,
                                  ws2)
    v1, r1, v2, r2 = host(vals), host(ranges), host(vals2), host(ranges2)
    assert int(host(counts)[0]) + int(host(counts2)[0]) == n_pairs
    for t in np.nonzero(r[:, 1] > r[:, 0])[0]:
        both = np.concatenate([v1[r1[t, 0]:r1[t, 1]], v2[r2[t, 0]:r2[t, 1]]])
        assert np.array_equal(both, v[r[t, 0]:r[t, 1]])
    # the prefix holds the nearest m Gaussians with a rectangle
    order = np.lexsort((np.arange(n), pr["depth32"].view(np.uint32)))
    order = order[(area > 0)[order] & pr["visible"][order]]
    near = np.zeros(n, dtype=bool)
    near[order[:m]] = True
    assert near[v1[: int(host(counts)[0])]].all() and not near[v2[: int(host(counts2)[0])]].any()
