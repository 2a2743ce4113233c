"""The dense build at mixed-basis sizes that are no multiple of 64 and with one
to three valence bands, against the FP64 oracle: every row count of the fused kernel's ragged form (one to six
64-row groups, one entry short of and past a group), one, two and three c c'
row blocks, and the shapes the unfused kernels keep (more than 384 entries,
five valence bands).

Tolerances (of max|H|): FP64 1e-12 (only the summation order differs); FP32
products accumulated over K = 2 Nmb terms, 2e-6.
"""
import numpy as np
import pytest

from oracle import bse as OB

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [  # (lattice, grid, nv, nc, nmb)
    ("cubic", (2, 2, 2), 1, 1, 1), ("cubic", (2, 2, 2), 2, 3, 15), ("hex", (3, 3, 1), 3, 4, 17),
    ("cubic", (3, 3, 3), 3, 2, 63), ("cubic", (2, 2, 2), 4, 5, 65), ("hex", (3, 3, 1), 2, 6, 127),
    ("hex", (5, 5, 1), 3, 4, 150), ("cubic", (2, 2, 2), 4, 4, 193), ("cubic", (2, 2, 2), 1, 6, 255),
    ("hex", (3, 3, 1), 4, 3, 257), ("cubic", (2, 2, 2), 2, 6, 319), ("cubic", (2, 2, 2), 3, 5, 321),
    ("hex", (3, 3, 1), 2, 2, 383), ("cubic", (2, 2, 2), 2, 3, 390), ("cubic", (2, 2, 2), 5, 2, 70),
    # several k in one column tile: whole and partial groups of k, straddled tiles
    ("cubic", (5, 5, 5), 1, 2, 64), ("hex", (7, 7, 1), 2, 5, 128), ("hex", (8, 8, 1), 3, 3, 192),
    ("cubic", (4, 4, 4), 1, 3, 33),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}{s[1][0]}_v{s[2]}c{s[3]}m{s[4]}")
@pytest.mark.parametrize("precname,tol", [("FP64", 1e-12), ("FP32", 2e-6)])
def test_ragged_build_matches_oracle(shape, precname, tol):
    import workloads
    from paper_2603_24860_amd import bse as B
    lattice, grid, nv, nc, nmb = shape
    cfg = dict(lattice=lattice, grid=grid, nv=nv, nc=nc, nmb=nmb, seed=11, name="t")
    print("[gpu-case] build", shape, precname, flush=True)
    S = workloads.device_system(cfg, getattr(B, precname))
    H = S.build()
    torch.cuda.synchronize()
    Ho = OB.hamiltonian(OB.make_problem(cfg))
    err = np.abs(H.cpu().numpy().astype(np.complex128) - Ho).max() / np.abs(Ho).max()
    assert err <= tol
