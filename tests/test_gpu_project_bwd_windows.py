"""The projection backward's windows (256, 512 or 1024 Gaussians a workgroup by
their number): a Gaussian's gradient does not depend on the window, so arrays
just above a limit give the bits of their part below it."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [131_072, 262_144])
@pytest.mark.parametrize("share", [0.0, 0.05, 1.0])
@pytest.mark.parametrize("accumulate", [False, True])
def test_windows_agree(n, share, accumulate):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    N = n + 1   # the larger window
    g = torch.Generator(device="cuda").manual_seed(3)
    p = torch.from_numpy(synth.gaussians(N, 4)).cuda()
    cam, rp = B.camera(synth.tetra_cameras()[0]), B.raster_params()
    radius = (torch.rand(N, device="cuda", generator=g) < 0.8).int() * 3
    clamp = torch.randint(0, 8, (N,), device="cuda", dtype=torch.uint8, generator=g)
    g2d = torch.randn((N, 9), device="cuda", generator=g)
    g2d[torch.rand(N, device="cuda", generator=g) >= share] = 0.0
    got = []
    for k in (n, N):
        grad = torch.full((B.PARAM_ROWS, k), 0.5, device="cuda")
        B.tgs_project_bwd(p[:, :k].contiguous(), k, cam, rp, radius[:k], clamp[:k], g2d[:k], grad,
                          accumulate=accumulate)
        got.append(grad)
    assert torch.equal(got[0], got[1][:, :n])
    live = (radius != 0) & (g2d != 0).any(1)
    assert bool((got[1][:, ~live] == (0.5 if accumulate else 0.0)).all())
    if share > 0:
        assert bool((got[1][:, live] != (0.5 if accumulate else 0.0)).any(0).all())
