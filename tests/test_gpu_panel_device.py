"""Which panels run in one launch on a device that holds few of their workgroups: the
number of workgroups that it is taken to hold is set from the host (96: 32 compute
units; 0: none at all), the launches are read from the library's profiler.  On the
device as it is every panel of up to 2304 trailing rows is one launch, on the default
stream, on a stream of its own and under capture.

Reference: the eigenvalues the matrix was made from, FP64 1e-11 of the norm (2).
"""
import contextlib
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n):
    """A banded Toeplitz matrix under a diagonal unitary: eigenvalues in closed form."""
    g = np.random.default_rng(n)
    ph = torch.from_numpy(np.exp(2j * np.pi * g.uniform(size=n)))
    a = torch.zeros((n, n), dtype=torch.complex128)
    i = torch.arange(n - 1)
    a[i, i + 1] = ph[:-1] * ph[1:].conj()
    a[i + 1, i] = a[i, i + 1].conj()
    b = torch.from_numpy(g.normal(size=n) + 1j * g.normal(size=n))
    return a.cuda(), b.cuda(), np.sort(2 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1)))


def _out(n):
    return [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]


@contextlib.contextmanager
def slots(n):
    from paper_2603_24860_amd import bse as B
    fn = B.lib.bse_eigh_panel_slots
    fn.restype, fn.argtypes = None, [ctypes.c_int64]
    fn(n)
    try:
        yield
    finally:
        fn(-1)


def _launches(run):
    from paper_2603_24860_amd import bse as B
    B.bse_prof_enable("k_")
    try:
        B.bse_prof_reset()
        run()
        torch.cuda.synchronize()
        return {k: c for k, (_, c) in B.bse_prof_collect().items()}
    finally:
        B.bse_prof_reset()
        B.bse_prof_enable(None)


def _panels(n, rows):
    """Panels in front of the tail (at most 96 rows), and those of at most `rows` rows."""
    j = [j for j in range(0, max(n - 96, 0), 32)]
    return len(j), sum(n - j0 - 1 <= rows for j0 in j)


@pytest.mark.parametrize("n", [97, 224, 225, 226, 720])
@pytest.mark.parametrize("held,rows", [(-1, 2304), (96, 192), (0, 0)])
def test_single(n, held, rows):
    from paper_2603_24860_amd import bse as B
    print("[gpu-case] panels of a device with", held, n, flush=True)
    a, b, lam = _case(n)
    ws = torch.full((B.bse_block_eigh_ws(n, 1, B.FP64, 0),), 255, dtype=torch.uint8, device="cuda")
    out = _out(n)
    with slots(held):
        seen = _launches(lambda: B.bse_block_eigh(a, b, B.FP64, *out, ws))
    every, one = _panels(n, rows)
    assert seen.get("k_panel", 0) == one
    assert seen.get("k_col0", 0) == every - one
    assert np.abs(out[0].cpu().numpy() - lam).max() <= 2e-11


@pytest.mark.parametrize("held,rows", [(-1, 2304), (96, 192), (0, 0)])
def test_batch(held, rows):
    from paper_2603_24860_amd import bse as B
    ns = [150, 720, 90, 97, 300, 226]
    print("[gpu-case] panels of a device with", held, ns, flush=True)
    H, b, lams = zip(*[_case(n) for n in ns])
    out = [_out(n) for n in ns]
    ws = torch.full((B.bse_batch_eigh_ws(ns, 1, B.FP64),), 255, dtype=torch.uint8, device="cuda")
    with slots(held):
        plan = B.bse_batch_eigh_plan(H, b, B.FP64, *zip(*out), ws)
    seen = _launches(lambda: B.bse_batch_eigh_run(plan))
    B.bse_batch_eigh_free(plan)
    # a panel index has a launch of either kind if any block takes it there
    col0 = one = 0
    for j0 in range(0, max(ns), 32):
        m = [n - j0 - 1 for n in ns if n - j0 > 96]
        col0 += any(x > rows for x in m)
        one += any(x <= rows for x in m)
    assert seen.get("k_col0", 0) == col0
    assert (seen.get("k_panel", 0) >= one) and bool(seen.get("k_panel")) == (one > 0)
    for o, lam in zip(out, lams):
        assert np.abs(o[0].cpu().numpy() - lam).max() <= 2e-11


def test_this_device():
    from paper_2603_24860_amd import bse as B
    n = 2305
    print("[gpu-case] panels of this device", n, flush=True)
    a, b, lam = _case(n)
    ws = torch.full((B.bse_block_eigh_ws(n, 1, B.FP64, 0),), 255, dtype=torch.uint8, device="cuda")
    every, one = _panels(n, 2304)
    assert every == one
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        out = _out(n)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            seen = _launches(lambda: B.bse_block_eigh(a, b, B.FP64, *out, ws))
        assert (seen.get("k_panel", 0), seen.get("k_col0", 0)) == (every, 0)
        assert np.abs(out[0].cpu().numpy() - lam).max() <= 2e-11
    # under capture: the same launches, so the same bits
    cap, graph = _out(n), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        B.bse_block_eigh(a, b, B.FP64, *cap, ws)
    graph.replay()
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(cap, out))
