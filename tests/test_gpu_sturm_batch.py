"""The bisection of one batched launch whose blocks lie on both sides of every line of
the rule that sets the lanes per eigenvalue (64 up to 1024 rows, 32 up to 2048, 16 up to
4096, 8 above), so that workgroups of different group widths run side by side.

Reference: the closed-form eigenvalues of the tridiagonal.  The reduction starts at e_1
and leaves the matrix as it is up to signs; the bisection is backward stable: 32 eps
sqrt(n) of the norm (2), and 8 eps32 sqrt(n) of it with FP32 storage.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precname", ["FP64", "FP32"])
@pytest.mark.parametrize("ns", [[1025, 96, 1024, 1, 700], [2048, 4097, 1024, 2049, 4096, 33]])
def test_blocks_of_every_group_width(ns, precname):
    from paper_2603_24860_amd import bse as B
    prec = getattr(B, precname)
    print("[gpu-case] sturm batch", ns, precname, flush=True)
    dt = torch.complex128 if prec == B.FP64 else torch.complex64
    H, b, out = [], [], []
    for n in ns:
        h = torch.zeros((n, n), dtype=dt, device="cuda")
        i = torch.arange(n - 1, device="cuda")
        h[i, i + 1] = h[i + 1, i] = 1.0
        H.append(h)
        b.append(torch.zeros(n, dtype=torch.complex128, device="cuda"))
        b[-1][0] = 1.0
        out.append([torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
                    for _ in range(3)])
    ws = torch.full((B.bse_batch_eigh_ws(ns, int(prec == B.FP64), prec),), 255, dtype=torch.uint8,
                    device="cuda")
    plan = B.bse_batch_eigh_plan(H, b, prec, *zip(*out), ws)
    B.bse_batch_eigh_run(plan)
    torch.cuda.synchronize()
    B.bse_batch_eigh_free(plan)
    for n, o in zip(ns, out):
        ref = np.sort(2 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1)))
        tol = 32 * 2.2e-16 if prec == B.FP64 else 8 * 6e-8
        assert np.abs(o[0].cpu().numpy() - ref).max() <= tol * np.sqrt(n) * 2, n
