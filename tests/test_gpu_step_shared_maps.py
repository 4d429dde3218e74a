"""Steps whose views share one error and age map: the updates run in turn."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared", ["both", "error", "age"])
def test_views_with_one_map(shared):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd.pipeline import StepConfig, Trainer
    W, H = 150, 107
    cams = [synth.look_at(eye, fx=180.0, fy=180.0, width=W, height=H) for eye in ((2.4, -1.1, 1.3), (-2.0, 1.5, 0.9))]
    gts = [torch.from_numpy(synth.image(H, W, k).astype(np.float32)).cuda() for k in range(2)]
    E = [torch.from_numpy(synth.error_map(H, W, 60 + k).view(np.int16)).cuda() for k in range(2)]
    A = [torch.from_numpy(synth.age_map(H, W, 70 + k).view(np.int16)).cuda() for k in range(2)]
    if shared in ("both", "error"):
        E[1] = E[0]
    if shared in ("both", "age"):
        A[1] = A[0]
    tr = Trainer(torch.from_numpy(synth.gaussians(2000, 8, logscale_mean=-3.0)).cuda(), cams, gts,
                 StepConfig(rate_permille=250, fuse_views=True), E=E, A=A)
    for _ in range(3):
        torch.cuda.synchronize()
        age = [a.cpu().numpy().astype(np.int64) for a in A]
        used = tr.step([0, 1])
        torch.cuda.synchronize()
        for k, vb in enumerate(used):   # age 0 where sampled, else one more, a view after the other
            hit = np.zeros((H, W), bool)
            off, pix = vb.tile_off.cpu().numpy(), vb.pix.cpu().numpy()
            for s, t in enumerate(vb.valid_tiles.cpu().numpy()):
                loc = pix[off[s]:off[s + 1]].astype(int)
                hit[t // vb.tiles_x * 16 + loc // 16, t % vb.tiles_x * 16 + loc % 16] = True
            for j in (0, 1) if shared in ("both", "age") else (k,):
                age[j] = np.where(hit, 0, age[j] + 1)
        for a, want in zip(A, age):
            assert np.array_equal(a.cpu().numpy(), want)
