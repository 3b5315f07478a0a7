"""HLLD with constrained transport, whose normal field is the face's own, in
every region of the fan: cells with independent random states and faces with
independent random fields (their divergence does not matter to a single
stage), against the oracle.  The bound is that of the stage on unrelated cells
with the cell-centred field: |dL| <= 6 faces x 2000 eps F / dx, F the largest
physical flux of the states, and two roundings of the stored state.
"""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W
from tests.test_gpu_hlld_regions import EPS, random_cells

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("emf", ["mean", "upwind"])
@pytest.mark.parametrize("riemann", ["hlld", "hll"])
def test_stage_on_unrelated_cells_and_faces(dtype, emf, riemann):
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = (67, 13, 11)
    setup = W.make_setup("random_cells", 3, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, glm=False)
    setup["ct"], setup["ct_emf"] = True, emf
    rng = np.random.default_rng(12)
    V = np.zeros((12, n[2], n[1], n[0]))
    V[:9] = random_cells(n, 11)
    V[9:] = rng.uniform(-1.5, 1.5, V[9:].shape) * rng.choice([0.0, 0.1, 1.0], V[9:].shape)
    o = C.Oracle(setup)
    np_t = np.float64 if dtype == "f64" else np.float32
    U0 = o.prim_to_cons(V).astype(np_t).astype(np.float64)  # the same state on both sides
    for d, ax in ((0, 2), (1, 1), (2, 0)):  # the cell field of the rounded faces
        U0[5 + d] = (0.5 * (U0[9 + d] + np.roll(U0[9 + d], -1, axis=ax))).astype(np_t)
    V = o.cons_to_prim(U0)
    assert V[4].min() > 0.1
    dt, ch = o.cfl(U0)
    dt *= 0.1
    _, u1 = o.step(U0, dt, ch, want_u1=True)

    ctx = Context(setup, dtype)
    Un = torch.from_numpy(U0.astype(np_t)).cuda()
    out, U1 = torch.empty_like(Un), torch.empty_like(Un)
    ctx.step(Un, out, dt, ch, U1_out=U1)
    torch.cuda.synchronize()

    vmax, bmax = np.abs(V[1:4]).max(), max(np.abs(V[5:8]).max(), np.abs(U0[9:]).max())
    flux = (U0[4].max() + V[4].max() + 1.5 * bmax ** 2) * vmax
    bound = 2 * EPS[dtype] * np.abs(U0).max() + 6 * 2000 * EPS[dtype] * flux * dt * max(n)
    err = np.abs(U1.double().cpu().numpy() - u1).max()
    change = np.abs(u1 - U0).max()
    print(f"{dtype} {emf} {riemann}: max error {err:.2e}, bound {bound:.2e}, largest change {change:.2e}", flush=True)
    assert err <= bound
    assert change > 100 * bound


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("riemann", ["hlld", "hll"])
def test_the_sign_of_a_zero_normal_field(dtype, riemann):
    """B_n = +0 and -0 (whose sign bit HLLD's masks read) and gas at rest with
    velocities of either zero: the same step and the same adjoint."""
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = 70
    setup = W.make_setup("zeros", 1, (n,), gamma=5.0 / 3.0, cfl=0.4, riemann=riemann, bc=W.OUTFLOW_X, glm=False)
    rng = np.random.default_rng(2)
    V = rng.uniform(0.5, 1.5, (9, 1, 1, n))
    V[1:4] = rng.uniform(-1.0, 1.0, (3, 1, 1, n)) * rng.choice([0.0, 1.0], n)
    V[5], V[8] = 0.0, 0.0
    ctx = Context(setup, dtype, adjoint=True)
    U = ctx.prim_to_cons(torch.from_numpy(V).cuda())
    dt, ch = ctx.cfl_dt(U)
    lam = torch.from_numpy(rng.normal(size=V.shape)).cuda()
    results = []
    for sign in (1.0, -1.0):
        Us = U.clone()
        Us[1:8][U[1:8] == 0] *= sign
        nxt, U1 = torch.empty_like(U), torch.empty_like(U)
        ctx.step(Us, nxt, dt, ch, 1.0, U1_out=U1)
        results.append((nxt, U1, ctx.step_adjoint(Us, U1, lam, torch.empty_like(lam), dt, ch, 1.0)))
    for a, b in zip(*results):
        assert torch.isfinite(a).all()
        assert torch.equal(a, b)  # (+0 equals -0)
    ctx.close()
