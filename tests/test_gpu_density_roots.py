"""The distances of the density sums, fused in the backward and by the walk of
their own: with one sample every Gaussian's sums have one term, and the two
kernels give the same bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mpt", [64, 128, 256])
def test_fused_distance_bits(mpt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    n = 3000
    rng = np.random.default_rng(9)
    rec = np.zeros((n, 12), np.float32)
    xy = rng.uniform(-9, 25, (2, n))
    rec[:, 0], rec[:, 1] = np.floor(xy)
    rec[:, 2:4] = (xy - np.floor(xy)).T
    rec[:, 4], rec[:, 5], rec[:, 6] = 10 ** rng.uniform(-4, -1, n), rng.normal(0, 0.5, n), 10 ** rng.uniform(-4, -1, n)
    rec[:, 7] = rng.uniform(0.005, 0.012, n)   # faint: the walk passes the whole list
    rec[:, 8:11] = rng.uniform(0, 1, (n, 3))
    i32 = dict(dtype=torch.int32, device="cuda")
    args = (torch.from_numpy(rec).cuda(), torch.arange(n, **i32), torch.tensor([[0, n]], **i32), 1, 1, 16, 16,
            torch.zeros(1, **i32), torch.tensor([0, 1], **i32), torch.tensor([119], dtype=torch.uint8, device="cuda"),
            1, mpt, B.raster_params())
    out, nc = torch.empty((1, 4), device="cuda"), torch.empty(1, **i32)
    B.tgs_render_fwd(*args, out, nc, None, None)
    err, dl = torch.full((1,), 0.7, device="cuda"), torch.full((1, 4), 0.01, device="cuda")
    fused, walk = torch.zeros((n, 4), device="cuda"), torch.zeros((n, 4), device="cuda")
    B.tgs_render_bwd_density(*args, out, nc, dl, torch.zeros((n, 9), device="cuda"), err, n, fused)
    B.tgs_density_accumulate(*args, nc, err, n, walk)
    a, b = fused[:, :3].cpu().numpy(), walk[:, :3].cpu().numpy()
    assert (b[:, 2] > 0).sum() > 500
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
