"""Panels given up as a joint effort: one workgroup runs every workgroup's part, with
the same bits.  The host makes the count of arrivals start below zero, so that the
workgroups of every panel wait their 20 ms in vain and every kernel ends normally.
Sizes: one row and one workgroup past the tail, the switch from two to
three rows per wave (1536 trailing rows), the largest panel (2304) and the first size
whose leading panel is too large, with and without kept reflectors; a batch; and more
single-launch panels at once than the device holds.

Each result is compared bit for bit with the joint run, which is checked against the
eigenvalues the matrix was made from (FP64 1e-11 of the norm, 2).
"""
import contextlib
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n):
    """A Toeplitz matrix of bandwidth one under a reflection: dense, eigenvalues in closed form."""
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.view_as_complex(torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g))
    v /= torch.linalg.norm(v)
    a = torch.zeros((n, n), dtype=torch.complex128, device="cuda")
    i = torch.arange(n - 1, device="cuda")
    a[i, i + 1] = a[i + 1, i] = 1.0
    a -= 2 * torch.outer(v, v.conj() @ a)
    a -= 2 * torch.outer(a @ v, v.conj())
    a = (a + a.conj().T.contiguous()) / 2
    b = torch.view_as_complex(torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g))
    return a, b, np.sort(2 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1)))


def _out(n):
    return [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]


@contextlib.contextmanager
def absent(wgs):
    from paper_2603_24860_amd import bse as B
    fn = B.lib.bse_eigh_panel_absent
    fn.restype, fn.argtypes = None, [ctypes.c_int32]
    fn(wgs)
    try:
        yield
    finally:
        fn(0)


def _ws(n, k=0):
    from paper_2603_24860_amd import bse as B
    return torch.full((B.bse_block_eigh_ws(n, 1, B.FP64, k),), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n,k", [(97, 0), (104, 0), (105, 3), (129, 0), (333, 0), (720, 10),
                                 (1536, 0), (1537, 0), (1538, 0), (1570, 5), (2304, 0), (2305, 0),
                                 (2306, 0)])
def test_single(n, k):
    from paper_2603_24860_amd import bse as B
    print("[gpu-case] panel given up", n, k, flush=True)
    a, b, lam = _case(n)
    ref = _out(n)
    B.bse_block_eigh(a, b, B.FP64, *ref, _ws(n, k), nrefine=k)
    assert np.abs(ref[0].cpu().numpy() - lam).max() <= 2e-11
    out = _out(n)
    with absent(1):
        B.bse_block_eigh(a, b, B.FP64, *out, _ws(n, k), nrefine=k)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(out, ref))


def test_batch():
    from paper_2603_24860_amd import bse as B
    ns = [300, 90, 1600, 97, 700, 300]
    print("[gpu-case] panels of a batch given up", ns, flush=True)
    H, b, lams = zip(*[_case(n) for n in ns])
    got = []
    for missing in (0, 1):
        out = [_out(n) for n in ns]
        ws = torch.full((B.bse_batch_eigh_ws(ns, 1, B.FP64),), 255, dtype=torch.uint8, device="cuda")
        with absent(missing):
            plan = B.bse_batch_eigh_plan(H, b, B.FP64, *zip(*out), ws)
        for _ in range(2):
            B.bse_batch_eigh_run(plan)
        torch.cuda.synchronize()
        B.bse_batch_eigh_free(plan)
        got.append([x for o in out for x in o])
    for o, lam in zip(got[0][::3], lams):
        assert np.abs(o.cpu().numpy() - lam).max() <= 2e-11
    assert all(torch.equal(x, y) for x, y in zip(*got))


def test_more_panels_at_once_than_the_device_holds():
    """Eight FP64 solves of 1500 rows and more (each panel up to 192 workgroups, 768 fit) on
    eight streams: each equals its solve alone bitwise."""
    from paper_2603_24860_amd import bse as B
    jobs = []
    for n in (1500, 2305, 2000, 1633, 2200, 1535, 2305, 1800):
        a, b, _ = _case(n)
        ws, ref = _ws(n), _out(n)
        B.bse_block_eigh(a, b, B.FP64, *ref, ws)
        torch.cuda.synchronize()
        jobs.append((n, a, b, ws, ref, _out(n), torch.cuda.Stream()))
    for rep in range(2):
        print("[gpu-case] panels of eight streams", rep, flush=True)
        torch.cuda.synchronize()
        for n, a, b, ws, _, out, s in jobs:
            with torch.cuda.stream(s):
                B.bse_block_eigh(a, b, B.FP64, *out, ws)
        torch.cuda.synchronize()
        for n, _, _, _, ref, out, _ in jobs:
            assert all(torch.equal(x, y) for x, y in zip(out, ref)), n
