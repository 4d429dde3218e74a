"""tgs_project_views against tgs_project, view by view and bit for bit: one
view, the views of one launch (8) and more, counts around a wave and a
workgroup, every SH degree, with and without the gradient clear."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


def _outputs(B, n):
    d = dict(device="cuda")
    return [torch.full((n, 12), -7.0, **d), torch.full((n,), -7.0, **d),
            torch.full((n,), -7, dtype=torch.int32, **d), torch.full((n, 4), -7, dtype=torch.int32, **d),
            torch.full((n,), 7, dtype=torch.uint8, **d), torch.full((n, 9), 7.0, **d)]


@pytest.mark.parametrize("n,views,deg", [(1, 1, 3), (63, 2, 3), (64, 3, 0), (65, 8, 1), (256, 9, 2), (257, 10, 3),
                                         (5000, 17, 3), (1000, 0, 3)])
def test_views_equal_single_projections(B, n, views, deg):
    p = torch.from_numpy(synth.gaussians(n, 3, extent=2.5)).cuda()
    cams = [synth.look_at((3.0 * np.cos(k), 3.0 * np.sin(k), 0.3 * (k % 5) - 0.4), fx=200.0 + 10 * k, fy=210.0,
                          width=160 + 16 * k, height=131 + k) for k in range(views)]
    cams = [B.camera(c) for c in cams]
    rp = B.raster_params(sh_degree=deg)
    got = [_outputs(B, n) for _ in cams]
    clear = [o[5] if k % 3 != 1 else None for k, o in enumerate(got)]
    B.tgs_project_views(p, n, cams, rp, *[[o[j] for o in got] for j in range(5)], clear)
    for k, c in enumerate(cams):
        want = _outputs(B, n)
        B.tgs_project(p, n, c, rp, *want[:5], want[5] if clear[k] is not None else None)
        torch.cuda.synchronize()
        for j, (a, b) in enumerate(zip(got[k], want)):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (k, j)


def test_refuses_bad_arguments(B):
    p = torch.from_numpy(synth.gaussians(8, 3)).cuda()
    cam = B.camera(synth.tetra_cameras()[0])
    o = _outputs(B, 8)
    off = torch.empty(8 * 12 + 1, device="cuda")[1:].view(8, 12)
    rp = B.raster_params()
    for splat, c in ((None, cam), (off, cam)):
        with pytest.raises(RuntimeError):
            B.tgs_project_views(p, 8, [c], rp, [splat], [o[1]], [o[2]], [o[3]], [o[4]], [o[5]])
    bad = B.camera(synth.tetra_cameras()[0])
    bad.width = 0
    with pytest.raises(RuntimeError):
        B.tgs_project_views(p, 8, [cam, bad], rp, [o[0]] * 2, [o[1]] * 2, [o[2]] * 2, [o[3]] * 2, [o[4]] * 2,
                            [o[5]] * 2)
