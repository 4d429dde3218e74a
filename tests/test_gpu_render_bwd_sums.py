"""The backward's nine sums over a tile's samples, term by term.

With one sample per launch every sum has one term, so the opacity gradient is
that pixel's q itself and the others must be its products with the pixel's own
offset, to the roundings of those products.  With all samples in one launch
each sum must be that of the terms.  Splats much smaller than the tile at its
corner and its centre, and one whose centre lies 76,000 pixels away."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24   # half a unit in the last place: the error of one FP32 rounding
W, H, TILE = 16, 176, 10   # one column of tiles; the last one is rendered
# (a, beta, delta) of the conic and the centre, in image pixels
CASES = {
    "corner": [(2.9, 0.1, 2.5, 0.43, 160.31), (1.7, -0.4, 3.1, 1.06, 161.52)],
    "far_corner": [(3.3, 0.0, 3.3, 14.97, 174.52)],
    "centre": [(0.6, 0.3, 0.4, 7.61, 167.27), (0.05, -1.2, 0.3, 6.12, 169.88)],
    "thin": [(0.8, 3.7, 0.002, 9.41, 166.13)],
    "far": [(1e-7, -15.75681, 1e-8, 76028.55262, 4990.51823)],
}


def records(case):
    c = CASES[case]
    r = np.zeros((len(c), 12), np.float32)
    for i, (a, beta, delta, x, y) in enumerate(c):
        r[i] = [np.floor(x), np.floor(y), x - np.floor(x), y - np.floor(y), a, beta, delta, 0.61 - 0.2 * i,
                0.3 + 0.1 * i, 0.6, 0.8 - 0.3 * i, 1.0 + i]
    return r


def run(B, rec, locs, grad, mpt, scale=1.0):
    d = torch.device("cuda")
    n, P = len(rec), len(locs)
    i32 = dict(dtype=torch.int32, device=d)
    splat, vals = torch.from_numpy(rec).cuda(), torch.arange(n, **i32)
    ranges = torch.zeros((H // 16, 2), **i32)
    ranges[TILE, 1] = n
    args = (splat, vals, ranges, 1, H // 16, W, H, torch.tensor([TILE], **i32), torch.tensor([0, P], **i32),
            torch.tensor(locs, dtype=torch.uint8, device=d), 1, mpt, B.raster_params())
    out, nc = torch.empty((P, 4), device=d), torch.empty(P, **i32)
    B.tgs_render_fwd(*args, out, nc, None, None)
    dl = torch.zeros((P, 4), device=d)
    dl[:, :3] = torch.from_numpy(grad[locs]).cuda() * scale
    g = torch.zeros((n, 9), device=d)
    B.tgs_render_bwd(*args, out, nc, dl, g)
    return g.cpu().numpy().astype(np.float64)


def terms(rec, loc, q):
    """The geometric gradients of one pixel whose opacity gradient is q, and the
    size of what is added in each."""
    x0, y0 = np.float32(0), np.float32(16 * TILE)
    gx, gy = (rec[:, 0] - x0) + rec[:, 2], (rec[:, 1] - y0) + rec[:, 3]   # FP32, as staged
    dx, dy = (np.float32(loc % 16) - gx).astype(np.float64), (np.float32(loc // 16) - gy).astype(np.float64)
    a, beta, delta, o = rec[:, 4:8].astype(np.float64).T
    b = (rec[:, 5] * rec[:, 4]).astype(np.float64)
    c = delta + beta * b
    t = [o * (a * dx + b * dy) * q, o * (b * dx + c * dy) * q, -0.5 * o * q * dx * dx, -o * q * dx * dy,
         -0.5 * o * q * dy * dy]
    s = [o * (abs(a * dx) + abs(b * dy)) * abs(q), o * (abs(b * dx) + abs(c * dy)) * abs(q)]
    return np.stack(t, 1), np.stack(s + [abs(v) for v in t[2:]], 1)


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding
    binding.lib()
    return binding


# 64, 128 and 256 threads per tile
@pytest.mark.parametrize("mpt", [64, 128, 256])
@pytest.mark.parametrize("case", list(CASES))
def test_sums_are_the_terms(B, case, mpt):
    rec = records(case)
    rng = np.random.default_rng(3)
    grad = rng.normal(size=(256, 3)).astype(np.float32)
    locs = np.append(np.sort(rng.choice(255, mpt - 1, replace=False)), 255)   # the last one holds the far corner
    total, size, seen = np.zeros((len(rec), 9)), np.zeros((len(rec), 9)), 0
    for loc in locs:
        g = run(B, rec, [loc], grad, mpt)
        q = g[:, 5]
        t, s = terms(rec, loc, q)
        # q dx, (q dx) dx and the factor: three roundings; the centre also has
        # b = beta a, c = delta + beta b and the sum of its two products
        tol = np.concatenate([6 * ULP * s[:, :2], 4 * ULP * s[:, 2:]], 1)
        assert (np.abs(g[:, :5] - t) <= tol + 1e-36).all(), (loc, g[:, :5], t)
        total += g
        size[:, :5] += s
        size[:, 5:] += np.abs(g[:, 5:])
        seen += int((q != 0).sum())
    assert seen > 0
    g = run(B, rec, list(locs), grad, mpt)
    # a lane's four pixels, six folds, the waves, and the terms' own roundings
    assert (np.abs(g - total) <= (4 + 6 + 4 + 6) * ULP * size + 1e-36).all()


def test_overflow_stays_in_its_field(B):
    """A gradient so large that q d d^T overflows: the opacity's and the
    colours' sums, which do not, are those of a small gradient, scaled."""
    rec = records("far")
    grad = np.random.default_rng(4).normal(size=(256, 3)).astype(np.float32)
    locs = list(range(0, 256, 4))
    # a power of two that keeps q, but not q dx, within FP32's range
    a, b = run(B, rec, locs, grad, 64), run(B, rec, locs, grad, 64, 2.0 ** 118)
    assert not np.isfinite(b[:, :5]).all()
    assert (b[:, 5:] == a[:, 5:] * 2.0 ** 118).all()
