"""The tile pass's variants at the sizes where each begins and ends, against
the oracle bit for bit: chosen tiles, sample offsets and the tile map; one
tile, half of them and all but one drawn; few and many tiles without weight;
ragged last columns and rows with fewer pixels than samples, one row, one
column."""
import numpy as np
import pytest
import torch

from oracle import sampler

pytestmark = pytest.mark.gpu

# tiles across and down, image width and height short of them
GRIDS = [(1, 129, 3, 0), (128, 1, 0, 9), (32, 32, 0, 0), (41, 25, 15, 15), (128, 64, 5, 1), (2731, 3, 1, 14),
         (128, 128, 2, 0), (145, 113, 12, 7), (181, 182, 0, 3)]


@pytest.mark.parametrize("zero", [0.0, 0.6])
@pytest.mark.parametrize("TX,TY,dx,dy", GRIDS)
def test_tiles_bit_exact(TX, TY, dx, dy, zero):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    W, H, n_t, n_pix = 16 * TX - dx, 16 * TY - dy, TX * TY, 60
    rng = np.random.default_rng(n_t)
    pred = rng.lognormal(-2.0, 1.5, n_t).astype(np.float32)
    pred[rng.random(n_t) < zero] = 0.0
    E = torch.zeros((H, W), dtype=torch.int16, device="cuda")
    A = torch.zeros((H, W), dtype=torch.int16, device="cuda")
    w = np.minimum(16, W - 16 * (np.arange(n_t) % TX)) * np.minimum(16, H - 16 * (np.arange(n_t) // TX))
    keys = np.array(sampler.tile_race_keys(
        [int(np.floor(float(p) * int(a) * float(1 << 24))) for p, a in zip(pred, w)], 7, 3, 2), dtype=object)
    order = np.array(sorted(range(n_t), key=lambda t: (keys[t], t)))
    ws = torch.empty(B.tgs_sample_workspace_size(H, W), dtype=torch.uint8, device="cuda")
    for n_sel in (1, n_t // 2, n_t - 1):
        sp = B.sample_params(n_pix, n_tiles_sel=n_sel, seed=7, step=3, view=2)
        vt = torch.empty(n_sel, dtype=torch.int32, device="cuda")
        off = torch.empty(n_sel + 1, dtype=torch.int32, device="cuda")
        pix = torch.empty(n_sel * n_pix, dtype=torch.uint8, device="cuda")
        slot = torch.empty(n_t, dtype=torch.int32, device="cuda")
        totals = torch.zeros(2, dtype=torch.int64, device="cuda")
        B.tgs_sample(E, A, H, W, sp, vt, off, pix, slot, totals, ws, tile_pred=torch.from_numpy(pred).cuda())
        tiles = np.sort(order[:n_sel])
        want_off = np.concatenate([[0], np.cumsum(np.minimum(n_pix, w[tiles]))])
        want_slot = -np.ones(n_t, dtype=np.int64)
        want_slot[tiles] = np.arange(n_sel)
        assert np.array_equal(vt.cpu().numpy(), tiles), n_sel
        assert np.array_equal(off.cpu().numpy(), want_off), n_sel
        assert np.array_equal(slot.cpu().numpy(), want_slot), n_sel
        assert totals.tolist() == [int(want_off[-1]), n_sel]
