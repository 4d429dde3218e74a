"""Dense steps read no error or age maps: maps in host memory, strided maps or
none are accepted on every step."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("maps", ["none", "host", "strided"])
def test_dense_steps_leave_the_maps(maps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd.pipeline import StepConfig, Trainer
    W, H = 96, 64
    cams = [synth.look_at(eye, fx=110.0, fy=110.0, width=W, height=H) for eye in ((2.4, -1.1, 1.3), (-2.0, 1.5, 0.9))]
    gts = [torch.from_numpy(synth.image(H, W, k).astype(np.float32)).cuda() for k in range(2)]
    make = {"none": lambda: None,
            "host": lambda: [torch.ones((H, W), dtype=torch.int16) for _ in cams],
            "strided": lambda: [torch.ones((W, H), dtype=torch.int16, device="cuda").T for _ in cams]}[maps]
    E, A = make(), make()
    tr = Trainer(torch.from_numpy(synth.gaussians(800, 8, logscale_mean=-3.0)).cuda(), cams, gts,
                 StepConfig(rate_permille=None, fuse_views=True), E=E, A=A)
    losses = []
    for _ in range(3):
        losses.append(tr.loss_value(tr.step([0, 1])))
    tr.check_counts(wait_all=True)
    assert np.isfinite(losses).all() and losses[2] < losses[0]
    for m in (E or []) + (A or []):
        assert bool((m == 1).all())
