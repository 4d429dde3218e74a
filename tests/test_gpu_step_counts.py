"""A step's buffers keep their own pair counts after the slot moves on to
another set: a new Gaussian count, a new rate."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("change", ["densify", "rate"])
def test_counts_of_a_dropped_set(change):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd.pipeline import StepConfig, Trainer
    W, H, n = 96, 64, 800
    cams = [synth.look_at(eye, fx=110.0, fy=110.0, width=W, height=H) for eye in ((2.4, -1.1, 1.3), (-2.0, 1.5, 0.9))]
    gts = [torch.from_numpy(synth.image(H, W, k).astype(np.float32)).cuda() for k in range(2)]
    E = [torch.from_numpy(synth.error_map(H, W, 60 + k).view(np.int16)).cuda() for k in range(2)]
    A = [torch.from_numpy(synth.age_map(H, W, 70 + k).view(np.int16)).cuda() for k in range(2)]
    tr = Trainer(torch.from_numpy(synth.gaussians(n, 8, logscale_mean=-3.0)).cuda(), cams, gts,
                 StepConfig(rate_permille=250, fuse_views=True, density_stats=True), E=E, A=A)
    tr.step([0, 1])
    used = tr.step([0, 1])
    torch.cuda.synchronize()
    want = [int((vb.ranges[:, 1] - vb.ranges[:, 0]).sum()) for vb in used]
    if change == "densify":
        keep = torch.zeros(n, dtype=torch.uint8, device="cuda")
        keep[: n // 3] = 1
        tr.densify_and_prune(torch.zeros_like(keep), keep, torch.zeros((n, 3), device="cuda"), 0.0)
        later = tr.step([0, 1])
    else:
        later = tr.step([1, 0], rate_permille=500)
    torch.cuda.synchronize()
    assert all(a is not b for a, b in zip(used, later))
    assert [vb.n_pairs for vb in used] == want
    assert [vb.n_pairs for vb in later] == [int((vb.ranges[:, 1] - vb.ranges[:, 0]).sum()) for vb in later] != want
