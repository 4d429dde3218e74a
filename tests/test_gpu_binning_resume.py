"""tgs_bin_sort_resume_async after a call that did not fit: the lists, ranges,
keys and counts of a call with enough room, at both depth-order routes, over
grids of one group of strips and more, with tile subsets, after no and some
capacity, and again too small."""
import numpy as np
import pytest
import torch

import synth
from oracle import project
from oracle.params import RasterParams
from support import splat_record

pytestmark = pytest.mark.gpu

RP = RasterParams()


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n,size,share,cap1", [(257, (64, 64), None, 0), (3000, (640, 400), 0.4, 9),
                                               (16385, (300, 200), None, 1000), (700, (40, 4112), 0.5, 10),
                                               (500, (4100, 40), None, 10)])
def test_resumed_lists_equal(n, size, share, cap1):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    W, H = size
    p = synth.gaussians(n, 11, logscale_mean=-3.0)
    cam = synth.look_at((2.6, 0.4, 0.9), fx=1.1 * max(size), fy=1.1 * max(size), width=W, height=H)
    pr = project.project(p, cam, RP)
    TX, TY = pr["TX"], pr["TY"]
    slot = None
    if share is not None:
        slots = -np.ones(TX * TY, dtype=np.int32)
        keep = np.sort(np.random.default_rng(4).choice(TX * TY, int(share * TX * TY), replace=False))
        slots[keep] = np.arange(keep.size)
        slot = dev(slots)
    args = (dev(pr["rect"].T.astype(np.int32)), dev(splat_record(pr)), dev(pr["depth32"]), n, slot, TX, TY,
            RP.alpha_min)
    area = (pr["rect"][2] - pr["rect"][0]) * (pr["rect"][3] - pr["rect"][1])
    cap = int(area[pr["visible"]].sum()) + 3

    def outputs(c):
        return dict(keys=torch.full((max(c, 1),), -1, dtype=torch.int64, device="cuda"),
                    vals=torch.full((max(c, 1),), -1, dtype=torch.int32, device="cuda"), capacity=c,
                    ranges=torch.full((TX * TY, 2), -1, dtype=torch.int32, device="cuda"),
                    touched=torch.zeros(n, dtype=torch.uint8, device="cuda"),
                    counts=torch.zeros(2, dtype=torch.int64, device="cuda"),
                    ws=torch.empty(B.tgs_bin_sort_workspace_size(n, c, TX * TY), dtype=torch.uint8, device="cuda"))
    want, first, again, got = outputs(cap), outputs(cap1), outputs(cap1 + 5), outputs(cap)
    B.tgs_bin_sort_async(*args, **want)
    B.tgs_bin_sort_async(*args, **first)
    B.tgs_bin_sort_resume_async(*args, first["ws"], cap1, **again)   # still too small: empty lists
    assert int(again["counts"][1]) > cap1 + 5 and not bool(again["ranges"].any())
    B.tgs_bin_sort_resume_async(*args, first["ws"], cap1, **got)
    for name in ("counts", "ranges", "vals", "keys"):
        assert torch.equal(want[name], got[name]), name
    assert torch.equal(want["touched"], first["touched"])
