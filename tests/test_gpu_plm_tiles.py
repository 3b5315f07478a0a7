"""3D PLM stages at the edges of their 64 x 8 tiles and z chunks: grids one
cell below, at and above a tile, a single tile with many chunks, thin axes of
two cells (periodic wrap through the whole axis) and chunk lengths that leave
a remainder, with both boundary kinds, against the oracle.

Bounds as the parity tests': element-wise max|q - q_ref| / max|q_ref| <= 1e-8
(FP64) and 2e-4 (FP32), relative L1 <= 1e-10 and 1e-5 (two steps here).
"""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W
from tests.helpers import max_rel, rel_l1

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-5}
TOL_MAX = {"f64": 1e-8, "f32": 2e-4}
SHAPES = [(64, 8, 64), (63, 7, 65), (65, 9, 63), (2, 2, 2), (3, 2, 131), (130, 17, 2), (129, 16, 29)]


@pytest.mark.parametrize("n", SHAPES, ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc,limiter,order", [("periodic", "minmod", 2), ("outflow", "mc", 3)])
def test_tile_edges(n, dtype, bc, limiter, order):
    import torch

    from paper_2510_24175_amd.mhd import Context
    from paper_2510_24175_amd.rollout import advance

    setup = W.make_setup("tile_edges", 3, n, gamma=5.0 / 3.0, cfl=0.3, limiter=limiter, bc=((bc, bc),) * 3,
                         time_order=order)
    z, y, x = np.meshgrid(*[(np.arange(m) + 0.5) / m for m in n[::-1]], indexing="ij")
    V = np.empty((9, n[2], n[1], n[0]))
    for q in range(9):  # every component varies along every axis
        V[q] = 0.3 * np.sin(2 * np.pi * (x + 2 * y + 3 * z) + 0.7 * q) * np.cos(2 * np.pi * (x - y + z) + 0.3 * q)
    V[0] += 1.0
    V[4] += 1.0
    V[8] *= 0.1
    o = C.Oracle(setup)
    Uo, _, ho = o.run(o.prim_to_cons(V), nsteps=2)
    ctx = Context(setup, dtype)
    U, _, hist = advance(ctx, ctx.prim_to_cons(torch.from_numpy(V).cuda()), nsteps=2)
    Ug = U.double().cpu().numpy()
    assert rel_l1(Ug, Uo, ho[-1][1]).max() <= TOL[dtype]
    assert max_rel(Ug, Uo).max() <= TOL_MAX[dtype]
    _, _, sums = ctx.step_info()
    vol = np.abs(Uo[:9]).sum(axis=(1, 2, 3)) * ctx.cell_volume
    assert (np.abs(np.array(sums) - o.sums(Uo)) <= (1e-12 if dtype == "f64" else 1e-6) * vol.max()).all()
