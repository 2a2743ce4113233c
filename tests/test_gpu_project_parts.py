"""Projection with more than 18 bands, where the column bands are taken in parts:
two (19 to 21 bands on large cubic grids, from 33 bands on), three, and the sizes on
either side of the rule's lines (18 and 19, 21 and 22, 32 and 33 bands, calls too small to be
divided), H and seed pieces.

Reference: U^T H U in FP64 torch.  Tolerance: sums run in FP64, so FP64 results
differ by the summation order (1e-13 of max|H_mu|) and FP32 results by one rounding
of the result (2^-24 of it, 1e-7 of max|H_mu|).  A call that asks for every block
gives each the bits of a call with that block alone.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# the workgroups of 17 x 17 x 1, 8^3 and 6^3 are above the line, those of 4^3 below it
SHAPES = [("D6h", 17, 3, 7), ("D6h", 17, 2, 11), ("D6h", 17, 4, 6), ("D6h", 17, 5, 5),
          ("D6h", 17, 4, 8), ("D6h", 17, 3, 11), ("D6h", 17, 6, 6), ("D6h", 17, 6, 7),
          ("Oh", 6, 5, 6), ("Oh", 6, 6, 7), ("Oh", 4, 5, 6), ("Oh", 4, 6, 7), ("D6h", 7, 1, 40), ("Oh", 7, 3, 6), ("Oh", 8, 1, 19),
          ("Oh", 8, 3, 7)]


def _dense_u(host, nb):
    U = np.zeros((len(host["members"]), int(host["n"]) // nb))
    for o, r in enumerate(host["orb_dim"]):
        m = host["members"][host["mem_off"][o]:host["mem_off"][o + 1]]
        if r:
            u = host["ubasis"][host["ub_off"][o]:host["ub_off"][o] + len(m) * r]
            c = int(host["orb_off"][o]) // nb
            U[m, c:c + r] = u.reshape(-1, r)
    return torch.from_numpy(U).cuda()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}{s[1]}_{s[2] * s[3]}bands")
@pytest.mark.parametrize("dt,tol", [(torch.complex64, 1e-7), (torch.complex128, 1e-13)])
def test_parts(shape, dt, tol):
    from paper_2603_24860_amd import _lib, bse as B
    from paper_2603_24860_amd.system import DeviceBlock
    group, n1, nv, nc = shape
    grid = (n1, n1, n1 if group == "Oh" else 1)
    nb, nk = nv * nc, int(np.prod(grid))
    N = nk * nb
    print("[gpu-case] project parts", shape, dt, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    real = torch.float32 if dt == torch.complex64 else torch.float64
    pad = 3
    H = torch.view_as_complex(torch.randn((N, N + pad, 2), dtype=real, device="cuda",
                                          generator=g))[:, :N]
    Bv = torch.view_as_complex(torch.randn((N, 2), dtype=torch.float64, device="cuda", generator=g))
    names = [nm for nm, _, _ in B.bse_group_irreps(group)]
    blks = [b for b in (DeviceBlock(group, grid, nm, nv, nc) for nm in names) if b.n > 0]
    t = B.bse_dims_get(group, grid)
    p = _lib.Problem((ctypes.c_int32 * 3)(*grid), nv, nc, 1, t["nkorb"], t["ncls"], t["nkorb"])
    nan = float("nan")
    Hm = [torch.full((b.n, b.n + 1), nan, dtype=dt, device="cuda")[:, :b.n] for b in blks]
    Bm = [torch.full((b.n,), nan, dtype=torch.complex128, device="cuda") for b in blks]
    B.bse_project_blocks(p, H, Bv, [b.c for b in blks], Hm, Bm)
    torch.cuda.synchronize()
    act = "T1u" if group == "Oh" else "E1u"
    for b, hm, bm in zip(blks, Hm, Bm):
        if b.irrep not in (act, names[0]):
            assert not torch.isnan(torch.view_as_real(hm.contiguous())).any()
            continue
        one = torch.full((b.n, b.n), nan, dtype=dt, device="cuda")
        B.bse_project_blocks(p, H, Bv, [b.c], [one], [None])
        torch.cuda.synchronize()
        assert torch.equal(one, hm), b.irrep
        U = _dense_u(b.host, nb)  # [nk][r]: the bands are spectators
        r = U.shape[1]
        ref = torch.empty((b.n, b.n), dtype=torch.complex128, device="cuda")
        for part, out in ((H.real, ref.real), (H.imag, ref.imag)):
            rows = U.T.contiguous() @ part.double().reshape(nk, nb * N)
            cols = rows.view(r * nb, nk, nb).transpose(1, 2).reshape(-1, nk) @ U
            out.copy_(cols.view(r * nb, nb, r).transpose(1, 2).reshape(b.n, b.n))
        assert float((hm - ref).abs().max()) <= tol * float(ref.abs().max()), b.irrep
        bref = torch.complex(U.T @ Bv.real.reshape(nk, nb), U.T @ Bv.imag.reshape(nk, nb))
        assert float((bm - bref.reshape(-1)).abs().max()) <= 1e-13 * float(bref.abs().max())


@pytest.mark.parametrize("precname", ["FP32", "FP64"])
@pytest.mark.parametrize("lattice,grid,nc,irrep", [("hex", (12, 12, 1), 6, "E1u"),
                                                   ("cubic", (8, 8, 8), 5, "T1u")])
def test_parts_from_seed_pieces(precname, lattice, grid, nc, irrep):
    """The block from the pieces (24 bands: three parts, 20: two) is the projection of the H
    that the same pieces assemble, bit for bit."""
    import synth
    import workloads
    from paper_2603_24860_amd import bse as B
    prec = getattr(B, precname)
    print("[gpu-case] project parts seed", precname, grid, flush=True)
    S = workloads.device_system(dict(lattice=lattice, grid=grid, nv=4, nc=nc, nmb=64, seed=3,
                                     name="t"), prec)
    ws = torch.empty(B.bse_seed_ws(S.group, S.problem, prec), dtype=torch.uint8, device="cuda")
    plan = B.bse_seed_plan(S.group, S.problem, prec, ws)
    try:
        dt = torch.complex64 if prec == B.FP32 else torch.complex128
        H = torch.empty((S.N, S.N), dtype=dt, device="cuda")
        B.bse_build_seed(plan, H)
        blk = S.block(irrep)
        a, b = (torch.full((blk.n, blk.n), float("nan"), dtype=dt, device="cuda") for _ in range(2))
        B.bse_project_seed(plan, [blk.c], [a])
        B.bse_project_blocks(S.problem, H, None, [blk.c], [b], [None])
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    finally:
        B.bse_seed_free(plan)
