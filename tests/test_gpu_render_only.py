"""Buffers of a caller that only renders: the image is that of full buffers,
without the state record and gradients that a backward needs, and the error
maps' first render makes none either."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

W, H, N = 640, 480, 2000


def test_render_without_backward():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    from paper_2606_15924_amd.pipeline import StepConfig, Trainer, ViewBuffers
    cam = synth.look_at((2.4, -1.1, 1.3), fx=700.0, fy=700.0, width=W, height=H)
    p = torch.from_numpy(synth.gaussians(N, 8, logscale_mean=-3.0)).cuda()
    rp, state = B.raster_params(), B.tgs_render_state_size((W // 16) * (H // 16), 256)
    out = []
    for kw in ({}, {"backward": False}):
        at = torch.cuda.memory_allocated()
        vb = ViewBuffers(N, W, H, None, -1, "cuda", **kw)
        size = torch.cuda.memory_allocated() - at
        vb.project(p, B.camera(cam), rp)
        vb.bin_sort(alpha_min=rp.alpha_min)
        vb.render_fwd(rp)
        out.append((vb.out.clone(), vb.ncontrib.clone(), size))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][2] - out[1][2] >= state
    with pytest.raises(RuntimeError, match="without a backward"):
        vb.render_bwd(rp)

    gt = torch.from_numpy(synth.image(H, W, 0).astype(np.float32)).cuda()
    E = [torch.zeros((H, W), dtype=torch.int16, device="cuda")]
    A = [torch.zeros_like(E[0])]
    tr = Trainer(p, [cam], [gt], StepConfig(), E=E, A=A)
    del vb
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    at = torch.cuda.memory_allocated()
    tr.init_error_maps([0])
    assert torch.cuda.max_memory_allocated() - at < state
    want = torch.empty_like(E[0])
    B.tgs_error_init(out[0][0], gt, H, W, want)
    assert torch.equal(E[0], want)
