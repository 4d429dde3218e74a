"""The fused update's windows of consecutive Gaussians (64, 256 or 512 by
their number): a Gaussian's update does not depend on the window, so arrays
just above a limit give the bits of their part below it."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65_536, 262_144])
@pytest.mark.parametrize("flags", [None, 0.04, 0.9])
def test_windows_agree(n, flags):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    N = n + 1   # the larger window
    g = torch.Generator(device="cuda").manual_seed(3)
    p = torch.from_numpy(synth.gaussians(N, 4)).cuda()
    cams = [B.camera(c) for c in synth.tetra_cameras()[:2]]
    rp, op = B.raster_params(), B.optim_params()
    radius = [(torch.rand(N, device="cuda", generator=g) < 0.8).int() * 3 for _ in cams]
    clamp = [torch.randint(0, 8, (N,), device="cuda", dtype=torch.uint8, generator=g) for _ in cams]
    g2d = [torch.randn((N, 9), device="cuda", generator=g) * 1e-3 for _ in cams]
    touched = None if flags is None else (torch.rand(N, device="cuda", generator=g) < flags).to(torch.uint8)
    m0 = torch.randn((N, B.MOMENT_STRIDE), device="cuda", generator=g) * 1e-4
    v0 = torch.rand((N, B.MOMENT_STRIDE), device="cuda", generator=g) * 1e-6
    got = []
    for k in (n, N):
        q, m, v = p[:, :k].clone(memory_format=torch.contiguous_format), m0[:k].clone(), v0[:k].clone()
        ws = torch.empty(B.tgs_project_bwd_optimizer_views_workspace_size(k, len(cams)), dtype=torch.uint8, device="cuda")
        B.tgs_project_bwd_optimizer_step_views(q, k, cams, rp, [r[:k].contiguous() for r in radius],
                                               [c[:k].contiguous() for c in clamp], [x[:k].contiguous() for x in g2d],
                                               m, v, None if touched is None else touched[:k].contiguous(), op, 5, ws)
        got.append((q, m, v))
    (qa, ma, va), (qb, mb, vb) = got
    assert not torch.equal(qa, p[:, :n])
    assert torch.equal(qa, qb[:, :n]) and torch.equal(ma, mb[:n]) and torch.equal(va, vb[:n])
    assert bool(torch.isfinite(qb).all())
