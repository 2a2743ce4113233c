"""Workspaces of the size the eigensolvers asked for before the single-launch panels
(FP64 storage: without their exchange words; batches: without their launch tables)
are accepted, and the solve stays inside them.  Sizes as the library of that time
returned them; the larger one of today's query is accepted as well, and one 256 bytes
short of the former is refused.

Reference: the eigenvalues the matrices were made from (FP64 1e-11 of the norm, FP32
storage 8 eps32 sqrt(n)); the launches made are read from the library's profiler.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 4096


def _case(n, dt):
    """A banded Toeplitz matrix under a diagonal unitary: eigenvalues in closed form."""
    g = np.random.default_rng(n)
    ph = torch.from_numpy(np.exp(2j * np.pi * g.uniform(size=n)))
    a = torch.zeros((n, n), dtype=torch.complex128)
    i = torch.arange(n - 1)
    a[i, i + 1] = ph[:-1] * ph[1:].conj()
    a[i + 1, i] = a[i, i + 1].conj()
    b = torch.from_numpy(g.normal(size=n) + 1j * g.normal(size=n))
    return a.to(dt).cuda(), b.cuda(), np.sort(2 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1)))


def _out(n):
    return [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]


def _ws(size):
    return torch.full((size + GUARD,), 255, dtype=torch.uint8, device="cuda")


def _launches(run):
    from paper_2603_24860_amd import bse as B
    B.bse_prof_enable("k_")
    try:
        B.bse_prof_reset()
        run()
        torch.cuda.synchronize()
        return {k: c for k, (_, c) in B.bse_prof_collect().items() if c}
    finally:
        B.bse_prof_reset()
        B.bse_prof_enable(None)


@pytest.mark.parametrize("n,k,former", [(97, 0, 343808), (300, 20, 6013696), (720, 0, 9223424),
                                        (2400, 0, 96572928)])
def test_single(n, k, former):
    from paper_2603_24860_amd import _lib, bse as B
    print("[gpu-case] former workspace", n, k, flush=True)
    a, b, lam = _case(n, torch.complex128)
    for size, panels in ((former, False), (B.bse_block_eigh_ws(n, 1, B.FP64, k), True)):
        ws, out = _ws(size), _out(n)
        seen = _launches(lambda: B.bse_block_eigh(a, b, B.FP64, *out, ws[:size], nrefine=k))
        assert bool(seen.get("k_panel")) == panels
        assert np.abs(out[0].cpu().numpy() - lam).max() <= 2e-11
        assert bool((ws[size:] == 255).all())
    with pytest.raises(_lib.BseError) as e:
        B.bse_block_eigh(a, b, B.FP64, *out, ws[:former - 256], nrefine=k)
    assert e.value.status == _lib.EWORKSPACE


@pytest.mark.parametrize("ns,precname,former", [([162, 200, 97], "FP64", 2039296),
                                                ([162, 200, 97], "FP32", 1391616),
                                                ([720, 64, 720, 300], "FP64", 20499200),
                                                ([720, 64, 720, 300], "FP32", 11442432),
                                                ([2400, 130], "FP64", 97175040)])
def test_batch(ns, precname, former):
    from paper_2603_24860_amd import _lib, bse as B
    prec = getattr(B, precname)
    print("[gpu-case] former batch workspace", ns, precname, flush=True)
    fp64 = prec == B.FP64
    cases = [_case(n, torch.complex128 if fp64 else torch.complex64) for n in ns]
    H, bv, lams = zip(*cases)
    query = B.bse_batch_eigh_ws(ns, int(fp64), prec)
    for size, panels in ((former, False), (query, fp64)):
        ws, out = _ws(size), [_out(n) for n in ns]
        plan = B.bse_batch_eigh_plan(H, bv, prec, *zip(*out), ws[:size])
        try:
            seen = _launches(lambda: B.bse_batch_eigh_run(plan))
            assert bool(seen.get("k_panel")) == panels
            for n, o, lam in zip(ns, out, lams):
                tol = 2e-11 if fp64 else 16 * 6e-8 * np.sqrt(n)
                assert np.abs(o[0].cpu().numpy() - lam).max() <= tol
            B.bse_batch_eigh_config(plan, 2, 32)  # rewrites the launch tables
            B.bse_batch_eigh_run(plan)
            torch.cuda.synchronize()
            assert bool((ws[size:] == 255).all())
        finally:
            B.bse_batch_eigh_free(plan)
    with pytest.raises(_lib.BseError) as e:
        B.bse_batch_eigh_plan(H, bv, prec, *zip(*out), ws[:former - 256])
    assert e.value.status == _lib.EWORKSPACE
