"""HLLD and HLL fluxes in every region of the fan, on cells with independent
random states: supersonic interfaces of both signs, single- and double-star
regions on both sides of the contact, normal fields of both signs, and exact
zeros of the normal field and of the tangential field (the degenerate star
state).  The stage-1 state Un + dt L(Un) is compared with the oracle's on the
same state, along each axis.

Bound: a flux is about 200 operations on terms no larger than the largest
physical flux of the states, F; near-degenerate fans magnify their rounding,
for which a factor ten is allowed, so |dL| <= 6 faces x 2000 eps F / dx, and
the stored state adds two roundings of its own size.
"""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W

pytestmark = pytest.mark.gpu

EPS = {"f64": 2.0 ** -52, "f32": 2.0 ** -23}


def random_cells(n, seed):
    """Primitive cells with no relation between neighbours."""
    rng = np.random.default_rng(seed)
    shape = (n[2], n[1], n[0])
    V = np.zeros((9,) + shape)
    V[0] = rng.uniform(0.3, 3.0, shape)
    V[4] = rng.uniform(0.3, 3.0, shape)
    # a bulk velocity per cell of either sign, supersonic in a third of them
    mach = rng.choice([0.3, 1.0, 6.0], shape)
    V[1:4] = rng.uniform(-1.0, 1.0, (3,) + shape) * mach
    V[5:8] = rng.uniform(-1.5, 1.5, (3,) + shape) * rng.choice([0.0, 0.1, 1.0], (3,) + shape)
    V[8] = 0.05 * rng.uniform(-1.0, 1.0, shape)
    return V


@pytest.mark.parametrize("riemann", ["hlld", "hll"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("glm", [True, False])
def test_stage_on_unrelated_cells(dtype, riemann, glm):
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = (67, 13, 11)
    setup = W.make_setup("random_cells", 3, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, glm=glm)
    o = C.Oracle(setup)
    U0 = o.prim_to_cons(random_cells(n, 11))
    np_t = np.float64 if dtype == "f64" else np.float32
    U0 = U0.astype(np_t).astype(np.float64)  # the same state on both sides
    V = o.cons_to_prim(U0)
    dt, ch = o.cfl(U0)
    dt *= 0.1
    _, u1 = o.step(U0, dt, ch, want_u1=True)

    ctx = Context(setup, dtype)
    Un = torch.from_numpy(U0.astype(np_t)).cuda()
    out, U1 = torch.empty_like(Un), torch.empty_like(Un)
    ctx.step(Un, out, dt, ch, U1_out=U1)
    torch.cuda.synchronize()

    # largest term of the physical flux: (E + p_T)|v|, rho v^2 + p_T, |v||B|, c_h^2 |B|, psi
    vmax, bmax = np.abs(V[1:4]).max(), np.abs(V[5:8]).max()
    flux = max((U0[4].max() + V[4].max() + 1.5 * bmax ** 2) * vmax, ch * ch * bmax)
    bound = 2 * EPS[dtype] * np.abs(U0).max() + 6 * 2000 * EPS[dtype] * flux * dt * max(n)
    err = np.abs(U1.double().cpu().numpy() - u1).max()
    change = np.abs(u1 - U0).max()
    print(f"{dtype} {riemann} glm={glm}: max error {err:.2e}, bound {bound:.2e}, largest change {change:.2e}", flush=True)
    assert err <= bound
    assert change > 100 * bound
