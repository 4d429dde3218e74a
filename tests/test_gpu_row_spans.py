"""The binning's row intervals, element for element, against the same FP64
operations in the same order in numpy: random splats (thin, round, faint,
opaque, off the image, not positive definite) and splats whose extents end
exactly on tile boundaries, where an estimate could go to the wrong side."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TX, TY, TILE = 20, 14, 16
ALPHA_MIN = float(np.float32(1.0 / 255.0))


def expected(s):
    """Sorted (tile << 32 | id) of the splat records s, every rectangle the whole grid."""
    s = s.astype(np.float64)
    xi, yi, xf, yf, A, beta, delta, o = s[:, :8].T
    lia = math.log(1.0 / ALPHA_MIN)
    tau = math.ceil(128.0 * lia * 1.001) / 64.0
    with np.errstate(all="ignore"):
        t = np.where(o > 0, np.minimum(tau, np.ceil(64.0 * (2.0 * (np.log(o) + lia) + 0.004)) * (1.0 / 64.0)), -1.0)
        B = beta * A
        C = delta + beta * B
        det = A * delta
        pd = (A > 0) & (det > 0)
        ym = np.where(t > 0, np.sqrt((t * A) / det), -1.0)
        ys = np.where(t > 0, B * np.sqrt(t / (C * det)), 0.0)
        tA = t * A
        codes = []
        for y in range(TY):
            Y0, Y1 = (float(TILE * y) - yi) - yf, (float(TILE * y + TILE - 1) - yi) - yf
            ylo, yhi = np.maximum(Y0, -ym), np.minimum(Y1, ym)
            yr, yl = np.minimum(np.maximum(-ys, ylo), yhi), np.minimum(np.maximum(ys, ylo), yhi)
            sr = np.sqrt(np.maximum(0.0, tA - det * (yr * yr)))
            sl = np.sqrt(np.maximum(0.0, tA - det * (yl * yl)))
            PL = ((-sl - B * yl) / A + xf) + xi
            PR = ((sr - B * yr) / A + xf) + xi
            lo = np.minimum(np.maximum(np.ceil((PL - (TILE - 1)) * (1.0 / TILE)), 0), TX)
            hi = np.minimum(np.maximum(np.floor(PR * (1.0 / TILE)), -1), TX - 1)
            lo = np.where(pd, np.where(ylo <= yhi, lo, 0), 0)
            hi = np.where(pd, np.where(ylo <= yhi, hi, -1), TX - 1)
            for x in range(TX):
                ids = np.nonzero((lo <= x) & (x <= hi))[0]
                codes.append(((y * TX + x) << 32) | ids.astype(np.int64))
    return np.sort(np.concatenate(codes))


def splats(kind, n, rng):
    s = np.zeros((n, 12), dtype=np.float32)
    if kind == "boundaries":
        # round splats of standard deviation 2^k and t = 4 (or 1): extents 2^(k+1) (2^k) exactly
        k = rng.integers(0, 6, n)
        two = rng.random(n) < 0.5
        s[:, 4] = s[:, 6] = 0.25 ** k
        lia = math.log(1.0 / ALPHA_MIN)
        s[:, 7] = np.where(two, math.exp((255.5 / 64 - 0.004) / 2 - lia), math.exp((63.5 / 64 - 0.004) / 2 - lia))
        ext = np.where(two, 2.0 ** (k + 1), 2.0 ** k)
        sx, sy = rng.choice([-1.0, 1.0], n), rng.choice([-1.0, 1.0], n)
        s[:, 0] = 16 * rng.integers(0, TX + 1, n) + rng.choice([0, 15], n) + sx * ext
        s[:, 1] = 16 * rng.integers(0, TY + 1, n) + rng.choice([0, 15], n) + sy * ext
        return s
    sig1, sig2 = np.exp(rng.uniform(-1.5, 5.0, (2, n)))
    a = rng.uniform(0, math.pi, n)
    c, d = np.cos(a), np.sin(a)
    q00, q01, q11 = c * c / sig1**2 + d * d / sig2**2, c * d * (1 / sig1**2 - 1 / sig2**2), d * d / sig1**2 + c * c / sig2**2
    s[:, 0] = np.floor(rng.uniform(-100, 16 * TX + 100, n))
    s[:, 1] = np.floor(rng.uniform(-100, 16 * TY + 100, n))
    s[:, 2:4] = rng.random((n, 2))
    s[:, 4], s[:, 5] = q00, q01 / q00
    s[:, 6] = q11 - q01 * q01 / q00
    s[:, 7] = np.where(rng.random(n) < 0.1, rng.choice([0.0, 1e-3, 1.0 / 255, 1.0], n), rng.random(n))
    bad = rng.random(n) < 0.02
    s[bad, 6] *= rng.choice([-1.0, 0.0], bad.sum())
    return s


@pytest.mark.parametrize("kind,n", [("random", 20_000), ("boundaries", 20_000), ("random", 300)])
def test_row_intervals_bit_exact(kind, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    rng = np.random.default_rng(n + len(kind))
    s = splats(kind, n, rng)
    want = expected(s)
    cap = want.size + 64
    rect = torch.tensor([[0, 0, TX, TY]], dtype=torch.int32, device="cuda").repeat(n, 1)
    depth = torch.from_numpy(rng.uniform(0.5, 9.0, n).astype(np.float32)).cuda()
    vals = torch.zeros(cap, dtype=torch.int32, device="cuda")
    ranges = torch.zeros((TX * TY, 2), dtype=torch.int32, device="cuda")
    counts = torch.zeros(2, dtype=torch.int64, device="cuda")
    ws = torch.empty(B.tgs_bin_sort_workspace_size(n, cap, TX * TY), dtype=torch.uint8, device="cuda")
    B.tgs_bin_sort_async(rect, torch.from_numpy(s).cuda(), depth, n, None, TX, TY, 1.0 / 255.0, None, vals, cap, ranges,
                         None, counts, ws)
    assert counts.tolist() == [want.size] * 2
    r = ranges.cpu().numpy().astype(np.int64)
    tile = np.repeat(np.arange(TX * TY), r[:, 1] - r[:, 0])
    got = np.sort((tile << 32) | vals.cpu().numpy()[: want.size].astype(np.int64))
    assert np.array_equal(got, want)
