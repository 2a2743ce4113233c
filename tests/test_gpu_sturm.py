"""The eigenvalue step of bse_block_eigh on tridiagonals that strain its Sturm
sequence: exact splits with eigenvalues on the evaluation points, entries over
many orders of magnitude, very large and very small scales, and sizes around the
block length of the recurrence and the lanes per eigenvalue.

Reference: numpy eigvalsh in FP64.  Both sides are backward stable: 32 eps sqrt(n)
of the norm.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _tri(kind, n):
    r = np.random.default_rng(n)
    d, e = r.uniform(-2, 2, n), r.uniform(0.1, 1, max(n - 1, 0))
    if kind == "integers":       # diagonal: every off-diagonal exactly zero
        d, e = np.arange(n) % 9 - 4.0, e * 0
    elif kind == "splits":       # blocks of three, eigenvalues repeated exactly
        d, e = d * 0 + 1.0, np.where(np.arange(n - 1) % 3 == 2, 0.0, 1.0)
    elif kind == "graded":
        s = 10.0 ** (-np.arange(n) * (120.0 / n))
        d, e = d * s, e * np.sqrt(s[1:] * s[:-1])
    elif kind == "huge":
        d, e = d * 1e60, e * 1e60
    elif kind == "tiny":
        d, e = d * 1e-60, e * 1e-60
    return np.diag(d) + np.diag(e, 1) + np.diag(e, -1)


@pytest.mark.parametrize("kind", ["plain", "integers", "splits", "graded", "huge", "tiny"])
@pytest.mark.parametrize("n", [2, 8, 9, 10, 17, 90, 130, 700])
def test_eigenvalues(kind, n):
    from paper_2603_24860_amd import bse as B
    print("[gpu-case] sturm", kind, n, flush=True)
    T = _tri(kind, n)
    H = torch.from_numpy(T.astype(np.complex128)).cuda()
    b = torch.zeros(n, dtype=torch.complex128, device="cuda")
    b[0] = 1.0  # already e_1: the reduction leaves T as it is up to signs
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
    ws = torch.empty(B.bse_block_eigh_ws(n, 1, B.FP64, 0), dtype=torch.uint8, device="cuda")
    B.bse_block_eigh(H, b, B.FP64, *out, ws)
    torch.cuda.synchronize()
    ref = np.linalg.eigvalsh(T)
    tol = 32 * 2.2e-16 * np.sqrt(n) * max(np.abs(ref).max(), 1e-80)
    if kind == "tiny":  # the library's pivot guard and paddings scale with max(1, |T|)
        tol = 32 * 2.2e-16 * n
    assert np.abs(out[0].cpu().numpy() - ref).max() <= tol


@pytest.mark.parametrize("n", [1500, 2100, 4100, 8200])
def test_lanes_per_eigenvalue(n):
    """Sizes on either side of the rule that sets the lanes per eigenvalue, through the batched
    solver as well (FP64, one block): the same eigenvalues as numpy's on a tridiagonal."""
    from paper_2603_24860_amd import bse as B
    print("[gpu-case] sturm lanes", n, flush=True)
    old = B.bse_block_eigh_set_two_stage(1 << 40)
    try:
        k = np.arange(n)
        H = torch.zeros((n, n), dtype=torch.complex128, device="cuda")
        i = torch.arange(n - 1, device="cuda")
        H[i, i + 1] = H[i + 1, i] = 1.0
        b = torch.zeros(n, dtype=torch.complex128, device="cuda")
        b[0] = 1.0
        out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
        ws = torch.empty(B.bse_block_eigh_ws(n, 1, B.FP64, 0), dtype=torch.uint8, device="cuda")
        B.bse_block_eigh(H, b, B.FP64, *out, ws)
        torch.cuda.synchronize()
    finally:
        B.bse_block_eigh_set_two_stage(old)
    ref = np.sort(2 * np.cos(np.pi * (k + 1) / (n + 1)))
    assert np.abs(out[0].cpu().numpy() - ref).max() <= 32 * 2.2e-16 * np.sqrt(n) * 2
