"""The backward and the density walk in chunks on lists that end before, at and
past the start of the open-ended last chunk: the sums of one workgroup per tile.

A chunk's transmittances are those of the whole walk; the colour behind a
Gaussian, S, is taken from the recorded state where the whole walk carries it
along, so the two differ by the roundings of up to 1200 steps: 1200 * 2^-23 of
S, and so of the gradients' largest value."""
import numpy as np
import pytest
import torch

from support import assert_close

pytestmark = pytest.mark.gpu

W, H = 64, 32   # 8 tiles
N = 3000


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


def scene(B, mode):
    rng = np.random.default_rng(17)
    rec = np.zeros((N, 12), np.float32)
    xy = rng.uniform((-40, -40), (W + 40, H + 40), (N, 2))
    rec[:, :2], rec[:, 2:4] = np.floor(xy), xy - np.floor(xy)
    # wide and faint, so that every pixel composites nearly all of its list:
    # alpha 0.0045 to 0.006 over 1200 leaves T above 1e-3
    rec[:, 4], rec[:, 5], rec[:, 6] = 10 ** rng.uniform(-6, -5.3, N), rng.normal(0, 0.3, N), 10 ** rng.uniform(-6, -5.3, N)
    rec[:, 7] = rng.uniform(0.0047, 0.006, N)
    rec[:, 8:11] = rng.uniform(0, 1, (N, 3))
    last = (B.RENDER_CHUNKS + 2 * (2 ** (B.RENDER_LONG_CHUNKS - 1) - 1)) * B.RENDER_CHUNK_LEN
    lens = [last - 1, last, last + 1, last + 64, last + 65, 1200, last // 2, 1199]
    ends = np.cumsum(lens)
    vals = np.concatenate([np.sort(rng.choice(N, m, replace=False)) for m in lens])
    ranges = np.stack([ends - lens, ends], 1)
    i32 = dict(dtype=torch.int32, device="cuda")
    vt = off = pix = None
    n_st, mpt, P = 8, 256, W * H
    if mode != "dense":
        mpt = int(mode[6:])
        vt, off = torch.arange(8, **i32), torch.arange(0, 8 * mpt + 1, mpt, **i32)
        pix = torch.from_numpy(np.concatenate([np.sort(rng.choice(256, mpt, replace=False)) for _ in lens]).astype(np.uint8)).cuda()
        P = 8 * mpt
    args = (torch.from_numpy(rec).cuda(), torch.tensor(vals, **i32), torch.tensor(ranges, **i32), W // 16, H // 16, W, H,
            vt, off, pix, n_st, mpt, B.raster_params())
    state = torch.full((B.tgs_render_state_size(n_st, mpt) // 4,), float("nan"), device="cuda")
    out, nc = torch.empty((P, 4), device="cuda"), torch.empty(P, **i32)
    B.tgs_render_fwd(*args, out, nc, None, state)
    deep = (nc > last + 64).float().mean()
    assert 0.2 < float(deep) < 0.4 and float((nc > last).float().mean()) > 0.5   # two tiles of eight; five
    gen = torch.Generator(device="cuda").manual_seed(5)
    dl = torch.randn((P, 4), generator=gen, device="cuda") * 1e-3
    err = torch.rand(P, generator=gen, device="cuda")
    return args, out, nc, dl, err, state, (vals, ranges)


def close(got, want, what):
    a, b = got.cpu().numpy(), want.cpu().numpy()
    assert np.isfinite(a).all()
    assert_close(a, b, 1e-5, 1200 * 2.0 ** -23 * (np.abs(b).max(axis=0) + 1e-12), what)


@pytest.mark.parametrize("mode", ["sparse64", "sparse128", "sparse200", "dense"])
def test_chunks_past_the_last_start(B, mode):
    args, out, nc, dl, err, state, _ = scene(B, mode)
    g = [torch.zeros((N, 9), device="cuda") for _ in range(4)]
    s = [torch.zeros((N, 4), device="cuda") for _ in range(4)]
    B.tgs_render_bwd(*args, out, nc, dl, g[0])
    B.tgs_render_bwd(*args, out, nc, dl, g[1], state)
    close(g[1], g[0], "backward")
    B.tgs_render_bwd_density(*args, out, nc, dl, g[2], err, N, s[0])
    B.tgs_render_bwd_density(*args, out, nc, dl, g[3], err, N, s[1], state=state)
    close(g[3], g[0], "backward with density sums")
    close(s[1], s[0], "density sums in the backward")
    B.tgs_density_accumulate(*args, nc, err, N, s[2])
    B.tgs_density_accumulate(*args, nc, err, N, s[3], state=state)
    close(s[3], s[2], "density walk")
    close(s[1][:, :3], s[2][:, :3], "density sums, backward and walk")


@pytest.mark.parametrize("mode", ["sparse64", "dense"])
def test_deterministic_chunks(B, mode):
    args, out, nc, dl, _, state, (vals, ranges) = scene(B, mode)
    # ids ascend in every list: equal depths make that the lists' order
    depth = torch.ones(N, device="cuda")
    rect = torch.tensor([[0, 0, W // 16, H // 16]], dtype=torch.int32, device="cuda").repeat(N, 1)
    m = len(vals)
    g = [torch.zeros((N, 9), device="cuda") for _ in range(4)]
    ws = torch.empty(B.tgs_render_bwd_det_workspace_size(m, args[11], mode == "dense"), dtype=torch.uint8, device="cuda")
    B.tgs_render_bwd(*args, out, nc, dl, g[0])
    for k, st in ((1, None), (2, state), (3, state)):
        B.tgs_render_bwd_deterministic(*args, out, nc, dl, g[k], st, None, depth, rect, N, m, ws)
    close(g[1], g[0], "one workgroup per tile")
    close(g[2], g[0], "chunks")
    assert torch.equal(g[2], g[3])
