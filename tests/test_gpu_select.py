"""The k-th largest, one and two ranks at a time, against a sort of the order
keys: counts around a workgroup and a grid, equal values, signed zeros,
infinities, NaN, ranks at both ends and equal ranks."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def order_keys(bits):
    return np.where(bits & 0x80000000, ~bits, bits | 0x80000000).astype(np.uint32)


@pytest.mark.parametrize("kind", ["scores", "bits", "few", "equal"])
@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 4097, 300_001, 2_200_000])
def test_ranks_bit_exact(n, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_15924_amd import binding as B
    rng = np.random.default_rng(n)
    bits = {"scores": lambda: np.where(rng.random(n) < 0.7, 0.0, rng.lognormal(-3, 2, n)).astype(np.float32).view(np.uint32),
            "bits": lambda: rng.integers(0, 1 << 32, n, dtype=np.uint32),
            "few": lambda: rng.choice(np.array([0, 1 << 31, 0x7f800000, 0xff800000, 0x7fc00000, 0x3f800001], np.uint32), n),
            "equal": lambda: np.full(n, 0x3e800000, np.uint32)}[kind]()
    srt = np.sort(order_keys(bits))[::-1]
    v = torch.from_numpy(bits.view(np.float32)).cuda()
    ws = torch.empty(B.tgs_select_workspace_size(), dtype=torch.uint8, device="cuda")
    out = torch.empty(3, device="cuda")
    for k0, k1 in ((1, n), (n, 1), ((n + 1) // 2, (n + 1) // 2), (max(1, n // 5), max(1, n - n // 3))):
        B.tgs_select_kth_largest2(v, n, k0, k1, out[:2], ws)
        B.tgs_select_kth_largest(v, n, k1, out[2:], ws)
        got = order_keys(out.cpu().numpy().view(np.uint32))
        assert got.tolist() == [srt[k0 - 1], srt[k1 - 1], srt[k1 - 1]], (k0, k1)
    for bad in ((0, 1), (1, n + 1)):
        with pytest.raises((RuntimeError, ValueError)):
            B.tgs_select_kth_largest2(v, n, *bad, out[:2], ws)
