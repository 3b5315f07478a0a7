"""WENO-Z + SSP-RK3 at the edges of tiles and z chunks (GLM and constrained
transport with either edge EMF), and FP32 WENO-Z over jumps whose smoothness
indicators overflow.

Bounds as the parity tests': element-wise max|q - q_ref| / max|q_ref| <= 1e-8
(FP64) and 2e-4 (FP32), relative L1 <= 1e-10 and 1e-5 (one step here).
"""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W
from tests.helpers import max_rel, rel_l1

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-5}
TOL_MAX = {"f64": 1e-8, "f32": 2e-4}


@pytest.mark.parametrize("n", [(64, 8, 65), (65, 9, 131), (7, 4, 200)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("div", ["glm", "mean", "upwind"])
def test_chunk_edges(n, dtype, div):
    import torch

    from paper_2510_24175_amd.mhd import Context
    from paper_2510_24175_amd.rollout import advance

    setup, V = W.orszag_tang_3d(n) if div == "glm" else W.orszag_tang_3d_ct(n, emf=div)
    o = C.Oracle(setup)
    Uo, _, ho = o.run(o.prim_to_cons(V), nsteps=1)
    ctx = Context(setup, dtype)
    U, _, hist = advance(ctx, ctx.prim_to_cons(torch.from_numpy(V).cuda()), nsteps=1)
    Ug = U.double().cpu().numpy()
    assert rel_l1(Ug[:9], Uo[:9], ho[0][1]).max() <= TOL[dtype]
    assert max_rel(Ug[:9], Uo[:9]).max() <= TOL_MAX[dtype]


@pytest.mark.parametrize("q,jump", [(0, 1e6), (0, 1e12), (8, 1e12), (8, 1e18), (8, 1e21), (8, 1e30)])
def test_fp32_jumps_beyond_the_indicators_range(q, jump):
    """Squares of differences beyond 2e19 overflow in FP32 (psi with GLM off
    may jump by more); the step stays finite, and cells away from the jump
    keep their state up to the rounding of the two convex combinations of
    SSP-RK3 (1/3, 2/3 and 3/4, 1/4: at most an ulp each)."""
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = 64
    setup = W.make_setup("jump", 1, (n,), gamma=1.4, cfl=0.4, riemann="hlld", limiter="wenoz", bc=W.OUTFLOW_X,
                         time_order=3, glm=False)
    V = np.zeros((9, 1, 1, n))
    V[0], V[4], V[5], V[6] = 1.0, 1.0, 0.5, 0.25
    V[q, 0, 0, : n // 2] = jump
    ctx = Context(setup, "f32")
    U0 = ctx.prim_to_cons(torch.from_numpy(V).cuda())
    dt, ch = ctx.cfl_dt(U0)
    U = torch.empty_like(U0)
    ctx.step(U0, U, 1e-3 * dt, ch)
    torch.cuda.synchronize()
    bad = (~torch.isfinite(U)).sum().item()
    assert bad == 0
    for far in (slice(0, 20), slice(n - 20, n)):
        assert ((U - U0).abs()[..., far] <= 2 * 2.0 ** -23 * U0.abs()[..., far]).all()


# (HLL's product of a speed and the energy flux leaves the range at 1e6, 1e23)
@pytest.mark.parametrize("riemann,rho,p", [("hll", 1e10, 1e24), ("hll", 1e-24, 1e-13), ("hlld", 1e10, 1e24),
                                           ("hlld", 1e-24, 1e-13), ("hlld", 1e6, 1e23)])
def test_fp32_units_far_from_one(rho, p, riemann):
    """A smooth state in units whose pressure squared leaves the FP32 range:
    one step against the oracle, each component relative to its own scale."""
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = 64
    setup = W.make_setup("units", 1, (n,), gamma=5.0 / 3.0, cfl=0.4, riemann=riemann, bc=W.OUTFLOW_X)
    x = (np.arange(n) + 0.5) / n
    V = np.zeros((9, 1, 1, n))
    a, b = np.sqrt(p / rho), np.sqrt(p)
    V[0, 0, 0] = rho * (1 + 0.2 * np.sin(2 * np.pi * x))
    V[1, 0, 0] = 0.3 * a * np.cos(2 * np.pi * x)
    V[2, 0, 0] = 0.2 * a * np.sin(4 * np.pi * x)
    V[4, 0, 0] = p * (1 + 0.2 * np.cos(4 * np.pi * x))
    V[5] = 0.5 * b
    V[6, 0, 0] = 0.4 * b * np.sin(2 * np.pi * x + 0.4)
    o = C.Oracle(setup)
    U0 = o.prim_to_cons(V).astype(np.float32)
    dt, ch = o.cfl(U0.astype(np.float64))
    Uo = o.step(U0.astype(np.float64), dt, ch)
    ctx = Context(setup, "f32")
    Un = torch.from_numpy(U0).cuda()
    U = torch.empty_like(Un)
    ctx.step(Un, U, dt, ch)
    Ug = U.double().cpu().numpy()
    for q in (0, 1, 2, 4, 5, 6):
        assert np.abs(Ug[q] - Uo[q]).max() <= TOL_MAX["f32"] * np.abs(Uo[q]).max(), q
