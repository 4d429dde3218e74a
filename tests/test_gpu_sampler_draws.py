"""The sampler's draws within a tile at their limits, bit for bit against the
oracle: sample counts around multiples of a wave, ages with many ties and in
both bytes, weights that are zero, negative, infinite, NaN, subnormal and the
largest, tiles whose weight runs out, ragged edges."""
import numpy as np
import pytest
import torch

from oracle import sampler
from oracle.params import SampleParams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ages", ["ties", "wide", "top"])
@pytest.mark.parametrize("n_pix,hard,stable", [(1, 400, 300), (64, 1000, 0), (65, 0, 0), (129, 0, 1000),
                                               (200, 400, 300), (255, 500, 500), (256, 900, 100)])
def test_draws_bit_exact(n_pix, hard, stable, ages):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    W, H = 75, 53
    rng = np.random.default_rng(n_pix)
    E = rng.uniform(0.0, 1.0, (H, W)).astype(np.float16).view(np.uint16)
    E[rng.random((H, W)) < 0.3] = 0
    E[:16, :16] = 0                                    # no weight at all
    E[:16, 16:32] = 0
    E[3, 20] = 0x3c00                                  # one pixel of weight
    E[16:32, :16] = rng.integers(0, 1 << 16, (16, 16)) # any bit pattern
    E[16:32, 16:32] = rng.integers(1, 1 << 10, (16, 16))   # subnormal
    E[32:48, :16] = 0x7bff                             # the largest
    A = {"ties": lambda: rng.integers(0, 3, (H, W)), "wide": lambda: rng.integers(0, 1 << 16, (H, W)),
         "top": lambda: np.where(rng.random((H, W)) < 0.5, 65535, 255)}[ages]().astype(np.uint16)
    bsp = B.sample_params(n_pix, hard, stable, seed=9, step=4, view=1)
    n_st = B.tgs_sample_tile_count(H, W, bsp)
    n_t = ((W + 15) // 16) * ((H + 15) // 16)
    vt = torch.empty(n_st, dtype=torch.int32, device="cuda")
    off = torch.empty(n_st + 1, dtype=torch.int32, device="cuda")
    pix = torch.empty(n_st * n_pix, dtype=torch.uint8, device="cuda")
    slot = torch.empty(n_t, dtype=torch.int32, device="cuda")
    totals = torch.zeros(2, dtype=torch.int64, device="cuda")
    ws = torch.empty(B.tgs_sample_workspace_size(H, W), dtype=torch.uint8, device="cuda")
    B.tgs_sample(torch.from_numpy(E.view(np.int16)).cuda(), torch.from_numpy(A.view(np.int16)).cuda(), H, W, bsp, vt,
                 off, pix, slot, totals, ws)
    ref = sampler.sample_view(E, A, SampleParams(n_pix=n_pix, hard_permille=hard, stable_permille=stable), 9, 4, 1)
    g_off = off.cpu().numpy()
    assert np.array_equal(g_off, ref["tile_off"])
    assert np.array_equal(pix.cpu().numpy()[: g_off[-1]], ref["pix"])
