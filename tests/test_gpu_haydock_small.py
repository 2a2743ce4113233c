"""The Lanczos step of small FP32 blocks (k_hd_step_s: 2 <= n <= 2304, 16-byte aligned
rows) at the edges of its pairs, of its two forms (768), of the pairs it requests
ahead (1536) and of its range, with padded rows, against the oracle's plain Lanczos on the same
FP32-rounded matrix (bound of the other coefficient tests: 1e-10 of max|H| sqrt(n)).
The padding holds NaN: nothing past a row may be read into a sum.
"""
import math

import numpy as np
import pytest

from oracle import bse as OB

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 3, 8, 127, 128, 129, 767, 768, 769, 1535, 1537, 2047, 2303, 2304, 2305])
def test_small_block_steps(n):
    from paper_2603_24860_amd import bse as B
    print("[gpu-case] haydock small", n, flush=True)
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
    H = ((X + X.conj().T) / 2).astype(np.complex64).astype(np.complex128)
    b = rng.normal(size=n) + 1j * rng.normal(size=n)
    K = min(n, 20)
    ld = n + n % 2 + 6
    Hp = torch.full((n, ld), float("nan"), dtype=torch.complex64, device="cuda")
    Hp[:, :n] = torch.as_tensor(H, device="cuda").to(torch.complex64)
    Bt = torch.as_tensor(b, device="cuda")
    ga = torch.full((K,), float("nan"), dtype=torch.float64, device="cuda")
    gb = torch.full((K + 1,), float("nan"), dtype=torch.float64, device="cuda")
    ws = torch.full((B.bse_haydock_ws(n),), 255, dtype=torch.uint8, device="cuda")
    B.bse_haydock(Hp[:, :n], Bt, K, ga, gb, ws)
    torch.cuda.synchronize()
    ra, rb = OB.haydock_coefficients(H, b, K)
    scale = np.abs(H).max() * max(1.0, math.sqrt(n))
    assert np.abs(ga.cpu().numpy() - ra).max() <= 1e-10 * scale
    assert np.abs(gb.cpu().numpy()[:K] - rb[:K]).max() <= 1e-10 * max(scale, rb[0])
