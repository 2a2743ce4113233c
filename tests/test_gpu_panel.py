"""The single-launch panels of the block eigensolver (k_panel): sizes at the edges
of their rules (one panel, partial last workgroups, the switches of rows per
workgroup at 1536 trailing rows and to per-column launches above 2304), FP64
working storage (and FP32, which keeps per-column launches), with refinement (reflectors kept), many solves at once on
more streams than panels fit side by side, and a captured graph.

Reference: the eigenvalues the matrix was made from.  Tolerances: FP64 1e-11 of the
norm (the bound of the other eigensolver tests); FP32 storage rounds the working
copy once per panel, 8 eps32 sqrt(n) of the norm; bitwise where stated.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n, seed=0):
    g = torch.Generator(device="cuda").manual_seed(1000 * n + seed)
    z = torch.randn((n, n, 2), dtype=torch.float64, device="cuda", generator=g)
    q, _ = torch.linalg.qr(torch.view_as_complex(z).cpu())
    lam = np.sort(np.concatenate([np.repeat(np.linspace(-1, 1, n // 3), 3), np.ones(n % 3) * 1.5]))
    a = (q * torch.from_numpy(lam)) @ q.conj().T
    a = (a + a.conj().T) / 2
    b = torch.view_as_complex(torch.randn((n, 2), dtype=torch.float64, device="cuda", generator=g))
    return a.cuda(), b, lam


def _solver(B, a, b, prec, k=0):
    n = a.shape[0]
    H = a if prec == B.FP64 else a.to(torch.complex64)
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
    ws = torch.full((B.bse_block_eigh_ws(n, int(prec == B.FP64), prec, k),), 255,
                    dtype=torch.uint8, device="cuda")
    return (lambda: B.bse_block_eigh(H, b, prec, *out, ws, nrefine=k)), out


@pytest.mark.parametrize("n", [96, 97, 104, 128, 129, 161, 333, 1000, 1537, 1570])
@pytest.mark.parametrize("precname", ["FP64", "FP32"])
def test_panel_edges(n, precname):
    from paper_2603_24860_amd import bse as B
    prec = getattr(B, precname)
    print("[gpu-case] panel", n, precname, flush=True)
    a, b, lam = _case(n)
    run, out = _solver(B, a, b, prec)
    run()
    torch.cuda.synchronize()
    tol = 1e-11 if prec == B.FP64 else 8 * 6e-8 * np.sqrt(n)
    assert np.abs(out[0].cpu().numpy() - lam).max() <= tol * 1.5
    s = float(out[2].sum() / (b.abs() ** 2).sum())
    assert abs(s - 1) <= (1e-9 if prec == B.FP64 else 1e-5)


@pytest.mark.parametrize("n,precname,k", [(2306, "FP32", 0), (2350, "FP64", 0), (2400, "FP32", 0),
                                          (300, "FP32", 20), (1600, "FP64", 10)])
def test_panel_switch_and_refinement(n, precname, k):
    from paper_2603_24860_amd import bse as B
    prec = getattr(B, precname)
    print("[gpu-case] panel", n, precname, k, flush=True)
    g = np.random.default_rng(n)
    # a banded Toeplitz matrix under a diagonal unitary: eigenvalues in closed form
    lam = np.sort(2 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1)))
    ph = torch.from_numpy(np.exp(2j * np.pi * g.uniform(size=n))).cuda()
    a = torch.zeros((n, n), dtype=torch.complex128, device="cuda")
    i = torch.arange(n - 1, device="cuda")
    a[i, i + 1] = ph[:-1] * ph[1:].conj()
    a[i + 1, i] = a[i, i + 1].conj()
    b = torch.from_numpy(g.normal(size=n) + 1j * g.normal(size=n)).cuda()
    run, out = _solver(B, a, b, prec, k)
    run()
    torch.cuda.synchronize()
    om = out[0].cpu().numpy()
    tol = (1e-11 if prec == B.FP64 else 8 * 6e-8 * np.sqrt(n)) * 2
    assert np.abs(om - lam).max() <= tol
    if k:  # against the FP64 spectrum of the stored matrix
        H = (a if prec == B.FP64 else a.to(torch.complex64)).to(torch.complex128).cpu().numpy()
        ref = np.linalg.eigvalsh(H)[:k]
        assert np.abs(om[:k] - ref).max() <= 1e-9 * 2


def test_many_streams_at_once():
    """Eight solves on eight streams, several rounds: each equals its solve alone bitwise."""
    from paper_2603_24860_amd import bse as B
    jobs = []
    for j, (n, prec) in enumerate([(1500, B.FP32), (700, B.FP64), (1500, B.FP32), (300, B.FP64),
                                   (1200, B.FP32), (900, B.FP64), (162, B.FP64), (1000, B.FP32)]):
        g = torch.Generator(device="cuda").manual_seed(j)
        z = torch.view_as_complex(torch.randn((n, n, 2), dtype=torch.float64, device="cuda",
                                              generator=g))
        b = torch.view_as_complex(torch.randn((n, 2), dtype=torch.float64, device="cuda",
                                              generator=g))
        run, out = _solver(B, (z + z.conj().T) / 2, b, prec)
        run()
        torch.cuda.synchronize()
        jobs.append((run, out, [o.clone() for o in out], torch.cuda.Stream()))
    for rep in range(3):
        print("[gpu-case] panel streams", rep, flush=True)
        for run, out, _, _ in jobs:
            for o in out:
                o.fill_(float("nan"))
        torch.cuda.synchronize()
        for run, _, _, s in jobs:
            with torch.cuda.stream(s):
                run()
        torch.cuda.synchronize()
        for _, out, ref, _ in jobs:
            assert all(torch.equal(o, r) for o, r in zip(out, ref))


def test_captured_panels():
    """A captured solve replayed on changed input, with eager solves in between."""
    from paper_2603_24860_amd import bse as B
    n = 400
    a, b, _ = _case(n)
    run, out = _solver(B, a, b, B.FP64)
    run()
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run()
    for rep in range(4):
        print("[gpu-case] panel graph", rep, flush=True)
        a.mul_(1.25)
        a.diagonal().add_(0.125 * rep)
        run()
        torch.cuda.synchronize()
        ref = [o.clone() for o in out]
        for o in out:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, r) for o, r in zip(out, ref))


@pytest.mark.parametrize("scale", [1e-153, 1e-147, 1e-139])
@pytest.mark.parametrize("two_stage", [False, True])
def test_reflectors_near_underflow(two_stage, scale):
    """Couplings whose squares are denormal or barely normal: the reflectors of the
    panels and of the chase take the sequence without reciprocal estimates there."""
    from paper_2603_24860_amd import bse as B
    n = 140
    print("[gpu-case] tiny couplings", two_stage, scale, flush=True)
    g = np.random.default_rng(7)
    lam = np.sort(g.uniform(-1, 1, n))
    a = g.normal(size=(n, n)) + 1j * g.normal(size=(n, n))
    a = np.diag(lam).astype(complex) + scale * (a + a.conj().T)
    a, b = torch.from_numpy(a).cuda(), torch.from_numpy(g.normal(size=n) + 0j).cuda()
    nmin = B.bse_block_eigh_set_two_stage(2 if two_stage else 4096)
    try:
        run, out = _solver(B, a, b, B.FP64)
        run()
        torch.cuda.synchronize()
    finally:
        B.bse_block_eigh_set_two_stage(nmin)
    assert np.abs(out[0].cpu().numpy() - lam).max() <= 1e-11
