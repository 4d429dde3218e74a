"""tgs_bin_sort_views_async against the single-view calls, view by view:
lists, ranges, keys, counts and touched flags equal, at both depth-order
routes, over grids of different sizes (also ones that go one by one), tile
subsets, depth prefixes, five views (more than one batch) and a view whose
capacity is too small."""
import numpy as np
import pytest
import torch

import synth
from oracle import project
from oracle.params import RasterParams
from support import splat_record

pytestmark = pytest.mark.gpu

RP = RasterParams()
SIZES = [(640, 400), (48, 48), (2064, 96), (300, 512), (64, 64)]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def view(p, k, size, share):
    W, H = size
    cam = synth.look_at((2.6 - 0.2 * k, 0.4, 0.9), fx=1.1 * max(size), fy=1.1 * max(size), width=W, height=H)
    pr = project.project(p, cam, RP)
    n_t = pr["TX"] * pr["TY"]
    slot = None
    if share is not None:
        slots = -np.ones(n_t, dtype=np.int32)
        keep = np.random.default_rng(k).choice(n_t, max(1, int(share * n_t)), replace=False)
        slots[np.sort(keep)] = np.arange(keep.size)
        slot = dev(slots)
    area = (pr["rect"][2] - pr["rect"][0]) * (pr["rect"][3] - pr["rect"][1])
    return {"rect": dev(pr["rect"].T.astype(np.int32)), "splat": dev(splat_record(pr)), "depth": dev(pr["depth32"]),
            "slot": slot, "tx": pr["TX"], "ty": pr["TY"], "cap": int(area[pr["visible"]].sum()) + 3}


def outputs(B, v, n):
    n_t = v["tx"] * v["ty"]
    return {"keys": torch.full((v["cap"],), -1, dtype=torch.int64, device="cuda"),
            "vals": torch.full((v["cap"],), -1, dtype=torch.int32, device="cuda"),
            "ranges": torch.full((n_t, 2), -1, dtype=torch.int32, device="cuda"),
            "touched": torch.zeros(n, dtype=torch.uint8, device="cuda"),
            "counts": torch.zeros(3, dtype=torch.int64, device="cuda"),
            "ws": torch.empty(B.tgs_bin_sort_workspace_size(n, v["cap"], n_t), dtype=torch.uint8, device="cuda")}


@pytest.mark.parametrize("n,prefix,sizes,share", [
    (3000, -1, SIZES[:3], None), (3000, 700, SIZES, 0.4), (16385, -1, SIZES[:2], 0.5), (16385, 5000, SIZES[1:4], None),
    (257, -1, [(4100, 40), (640, 400)], None), (700, 200, [(40, 4112), (48, 48)], 0.5)])
def test_views_equal_single_calls(B, n, prefix, sizes, share):
    p = synth.gaussians(n, 11, logscale_mean=-3.0)
    views = [view(p, k, s, share if k % 2 == 0 else None) for k, s in enumerate(sizes)]
    views[1]["cap"] = 5   # this view's lists come out empty, the others whole
    want, got = ([outputs(B, v, n) for v in views] for _ in range(2))
    for v, o in zip(views, want):
        args = (v["rect"], v["splat"], v["depth"], n, v["slot"], v["tx"], v["ty"], RP.alpha_min)
        if prefix < 0:
            B.tgs_bin_sort_async(*args, o["keys"], o["vals"], v["cap"], o["ranges"], o["touched"], o["counts"],
                                 o["ws"])
        else:
            B.tgs_bin_sort_prefix_async(*args, prefix, o["keys"], o["vals"], v["cap"], o["ranges"], o["touched"],
                                        o["counts"], o["ws"])
    B.tgs_bin_sort_views_async([B.bin_view(v["rect"], v["splat"], v["depth"], v["slot"], v["tx"], v["ty"], o["keys"],
                                           o["vals"], v["cap"], o["ranges"], o["touched"], o["counts"], o["ws"])
                                for v, o in zip(views, got)], n, RP.alpha_min, prefix)
    torch.cuda.synchronize()
    assert int(want[0]["counts"][0]) > 0 and int(want[1]["counts"][1]) > 5
    for k, (w, g) in enumerate(zip(want, got)):
        for name in ("counts", "ranges", "vals", "keys", "touched"):
            assert torch.equal(w[name], g[name]), (k, name)
    # argument errors are reported before anything is queued, for any view
    bad = B.bin_view(views[0]["rect"], views[0]["splat"], views[0]["depth"], None, 0, 1, None, got[0]["vals"], 5,
                     got[0]["ranges"], None, got[0]["counts"], got[0]["ws"])
    with pytest.raises(RuntimeError):
        B.tgs_bin_sort_views_async([bad], n, RP.alpha_min, prefix)
    B.tgs_bin_sort_views_async([], n, RP.alpha_min, prefix)
