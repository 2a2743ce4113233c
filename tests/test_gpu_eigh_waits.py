"""Solves that cannot give eigenvalues say so: a wait of the bulge chase that runs out,
and a block that holds a NaN or an infinity (which is also what a word that never came
becomes in a single-launch panel).  Every eigenvalue is NaN, bse_block_eigh_status
reports n of them, and the next solve on the same workspace is as if nothing had
happened.  The wait is cut short from the host (it may not poll at all), so every
kernel leaves it as it would after a minute.
"""
import contextlib
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n, dt=torch.complex128):
    g = torch.Generator(device="cuda").manual_seed(n)
    z = torch.view_as_complex(torch.randn((n, n, 2), dtype=torch.float64, device="cuda", generator=g))
    b = torch.view_as_complex(torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g))
    return ((z + z.conj().T) / 2).to(dt).contiguous(), b


def _out(n):
    return [torch.full((n,), 7.0, dtype=torch.float64, device="cuda") for _ in range(3)]


@contextlib.contextmanager
def impatient():
    from paper_2603_24860_amd import bse as B
    fn = B.lib.bse_eigh_chase_impatient
    fn.restype, fn.argtypes = None, [ctypes.c_int32]
    fn(1)
    try:
        yield
    finally:
        fn(0)


@pytest.fixture
def solver(request):
    """One block, its reference solve, and a check of a solve that must fail."""
    from paper_2603_24860_amd import _lib, bse as B
    n, precname, k, two = request.param
    prec = getattr(B, precname)
    print("[gpu-case] no eigenvalues", request.node.name, flush=True)
    H, b = _case(n, torch.complex128 if prec == B.FP64 else torch.complex64)
    old = B.bse_block_eigh_set_two_stage(2 if two else 1 << 40)
    ws = torch.empty(B.bse_block_eigh_ws(n, int(prec == B.FP64), prec, k), dtype=torch.uint8,
                     device="cuda")

    def solve():
        out = _out(n)
        B.bse_block_eigh(H, b, prec, *out, ws, nrefine=k)
        return out

    def fails():
        bad = solve()
        with pytest.raises(_lib.BseError) as e:
            B.bse_block_eigh_status(n, prec, k, ws)
        assert e.value.status == _lib.ENOCONV
        assert B.bse_block_eigh_status(n, prec, k, ws, raise_on_noconv=False)[1] == n
        assert bool(torch.isnan(bad[0]).all())

    ref = solve()
    st = B.bse_block_eigh_status(n, prec, k, ws)
    assert st[1] == 0 and bool(torch.isfinite(ref[0]).all())
    yield H, fails
    out = solve()
    assert B.bse_block_eigh_status(n, prec, k, ws) == st
    assert all(torch.equal(x, y) for x, y in zip(out, ref))
    B.bse_block_eigh_set_two_stage(old)


@pytest.mark.parametrize("solver", [(300, "FP32", 0, True), (700, "FP64", 0, True),
                                    (700, "FP64", 10, True), (3000, "FP32", 0, True)], indirect=True)
def test_chase_wait_runs_out(solver):
    with impatient():
        solver[1]()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("solver", [(90, "FP64", 0, False), (300, "FP64", 0, False),
                                    (300, "FP32", 5, False), (1700, "FP64", 5, False),
                                    (700, "FP64", 0, True), (300, "FP32", 10, True)], indirect=True)
def test_block_not_finite(solver, value):
    H, fails = solver
    i, j = H.shape[0] // 2, H.shape[0] - 5  # met in the middle of the reduction
    keep = H[i, j].clone(), H[j, i].clone()
    H[i, j] = H[j, i] = value
    fails()
    H[i, j], H[j, i] = keep


def test_batch_not_finite():
    """Only the block that is not finite has no eigenvalues."""
    from paper_2603_24860_amd import bse as B
    ns = [400, 90, 300]
    print("[gpu-case] no eigenvalues, batch", ns, flush=True)
    H, b = zip(*[_case(n) for n in ns])
    got = []
    for value in (0.5, float("nan")):
        H[2][150, 150] = value
        ws = torch.empty(B.bse_batch_eigh_ws(ns, 1, B.FP64), dtype=torch.uint8, device="cuda")
        out = [_out(n) for n in ns]
        plan = B.bse_batch_eigh_plan(H, b, B.FP64, *zip(*out), ws)
        B.bse_batch_eigh_run(plan)
        torch.cuda.synchronize()
        B.bse_batch_eigh_free(plan)
        got.append([o[0] for o in out])
    for i, (ref, bad) in enumerate(zip(*got)):
        assert bool(torch.isfinite(ref).all())
        assert bool(torch.isnan(bad).all()) if i == 2 else torch.equal(ref, bad)
