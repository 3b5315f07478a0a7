"""2D and 1D stages over strips of tiles: one tile, a strip with a remainder,
a ragged last tile, two-cell axes, and every reduction path (FP32, FP64,
helper waves), against the oracle.  Bounds as the parity tests' (three steps
here); sums within 1e-12 (FP64) and 1e-6 (FP32) of the largest component's."""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W
from tests.helpers import max_rel, rel_l1

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-5}
TOL_MAX = {"f64": 1e-8, "f32": 2e-4}
SHAPES = [(64, 4), (65, 9), (2, 2), (130, 1031), (3, 517), (700, 8), (64,), (65,), (1000,)]


@pytest.mark.parametrize("n", SHAPES, ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("limiter,bc", [("minmod", "periodic"), ("wenoz", "outflow")])
def test_strips(n, dtype, limiter, bc):
    import torch

    from paper_2510_24175_amd.mhd import Context
    from paper_2510_24175_amd.rollout import advance

    setup = W.make_setup("strips", len(n), n, gamma=5.0 / 3.0, cfl=0.4, limiter=limiter, bc=((bc, bc),) * 3,
                         time_order=3 if limiter == "wenoz" else 2)
    nx, ny = n[0], (n[1] if len(n) > 1 else 1)
    y, x = np.meshgrid((np.arange(ny) + 0.5) / ny, (np.arange(nx) + 0.5) / nx, indexing="ij")
    if len(n) == 1:
        y = 0.25 * x
    V = np.empty((9, 1, ny, nx))
    for q in range(9):
        V[q, 0] = 0.25 * np.sin(2 * np.pi * (x + 2 * y) + 0.7 * q) * np.cos(2 * np.pi * (x - y) + 0.3 * q)
    V[0] += 1.0
    V[4] += 1.0
    V[8] *= 0.1
    o = C.Oracle(setup)
    Uo, _, ho = o.run(o.prim_to_cons(V), nsteps=3)
    ctx = Context(setup, dtype)
    U, _, hist = advance(ctx, ctx.prim_to_cons(torch.from_numpy(V).cuda()), nsteps=3)
    Ug = U.double().cpu().numpy()
    assert rel_l1(Ug, Uo, ho[-1][1]).max() <= TOL[dtype]
    assert max_rel(Ug, Uo).max() <= TOL_MAX[dtype]
    dt, ch, sums = ctx.step_info()
    dt1, ch1 = ctx.cfl_dt(U)
    assert (dt, ch) == (dt1, ch1)
    vol = np.abs(Uo).sum(axis=(1, 2, 3)) * ctx.cell_volume
    assert (np.abs(np.array(sums) - o.sums(Uo)) <= (1e-12 if dtype == "f64" else 1e-6) * vol.max()).all()
