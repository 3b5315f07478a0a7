"""Marching kernels over chunks of several planes (3D) or strips of several
tiles (2D), with a shorter last one: what a chunk carries from plane to plane
(register windows, z fluxes, the halo loaded ahead, the edge EMFs of two planes,
the reductions) against the oracle.  The shapes are thin, so that small grids
have more tiles than the device has places for workgroups.

march() restates the library's rule for the chunk length, so that each test
says which length and remainder it takes; it has to be kept in step with it.

Bounds as the parity tests': element-wise max|q - q_ref| / max|q_ref| <= 1e-8
(FP64) and 2e-4 (FP32), relative L1 <= 1e-10 and 1e-5 (two steps here), sums
within 1e-12 and 1e-6 of the largest component's.
"""
import numpy as np
import pytest

from oracle import coracle as C
from paper_2510_24175_amd import workloads as W
from tests.helpers import face_divergence, max_rel, rel_l1

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 1e-5}
TOL_MAX = {"f64": 1e-8, "f32": 2e-4}
TOL_SUM = {"f64": 1e-12, "f32": 1e-6}


def march(nx, ny, nz, rows, per_cu, warm, width=64):
    """(chunk length, number of chunks) along the last axis."""
    up = lambda a, b: -(-a // b)
    tiles = up(nx, width) * up(ny, rows)
    longest = min(nz, 64)
    most = max(4096, tiles * up(nz, longest))
    best = None
    for kz in range(longest, 0, -1):
        blocks = tiles * up(nz, kz)
        if blocks > most:
            break
        full, rest = divmod(blocks, 256 * per_cu)
        cost = (full + (0.2 + 0.8 * up(rest, 256) / per_cu if rest else 0.0)) * (kz + warm)
        if best is None or cost < best[0]:
            best = (cost, kz)
    return best[1], up(nz, best[1])


def stage_march(n, dtype, limiter):
    f32, weno = dtype == "f32", limiter == "wenoz"
    if len(n) == 2:
        rows = 8 if f32 and weno else 4
        return -(-n[1] // rows), march(n[0], 1, -(-n[1] // rows), 1, 1 if weno else (4 if f32 else 2),
                                       (1.0 if weno else 0.5) if f32 else 0.1)
    return n[2], march(*n, 4 if weno and not f32 else 8, 2 if f32 and not weno else 1, 2.0 if weno else 1.5)


def assert_several_planes(planes, plan, least):
    kz, chunks = plan
    print(f"{chunks} chunks of {kz}, {planes} planes", flush=True)
    assert kz >= least and chunks > 1 and planes % kz


def waves(n):
    """Primitives of which every component varies along every axis."""
    nx, ny, nz = (tuple(n) + (1,))[:3]
    z, y, x = np.meshgrid(*[(np.arange(m) + 0.5) / m for m in (nz, ny, nx)], indexing="ij")
    V = np.empty((9, nz, ny, nx))
    for q in range(9):
        V[q] = 0.25 * np.sin(2 * np.pi * (x + 2 * y + 3 * z) + 0.7 * q) * np.cos(2 * np.pi * (x - y + z) + 0.3 * q)
    V[0] += 1.0
    V[4] += 1.0
    V[8] *= 0.1
    return V


def check(setup, V, dtype):
    import torch

    from paper_2510_24175_amd.mhd import Context
    from paper_2510_24175_amd.rollout import advance

    o = C.Oracle(setup)
    Uo, _, ho = o.run(o.prim_to_cons(V), nsteps=2)
    ctx = Context(setup, dtype)
    U, _, _ = advance(ctx, ctx.prim_to_cons(torch.from_numpy(V).cuda()), nsteps=2)
    dt, ch, sums = ctx.step_info()
    dt_all, ch_all = ctx.cfl_dt(U)
    Ug = U.double().cpu().numpy()
    ctx.close()
    # 3D FP32 states: the fused maxima are of the cells an FP32 estimate picks, within its rounding
    near = 0.0 if dtype == "f64" or setup["ndim"] == 2 or setup.get("ct") else 2e-6
    assert abs(dt / dt_all - 1) <= near and abs(ch / ch_all - 1) <= near
    assert rel_l1(Ug[:9], Uo[:9], ho[-1][1]).max() <= TOL[dtype]
    assert max_rel(Ug[:9], Uo[:9]).max() <= TOL_MAX[dtype]
    vol = np.abs(Uo[:9]).sum(axis=(1, 2, 3)) * ctx.cell_volume
    assert (np.abs(np.array(sums) - o.sums(Uo)) <= TOL_SUM[dtype] * vol.max()).all()
    return o, Ug, Uo


@pytest.mark.parametrize("n", [(3, 515, 61), (17, 130, 61), (67, 65, 57), (130, 33, 69)],
                         ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc,limiter,riemann,order,glm", [
    ("periodic", "minmod", "hlld", 2, True), ("outflow", "mc", "hll", 3, False), ("outflow", "minmod", "hlld", 3, True),
    ("periodic", "wenoz", "hll", 2, True), ("outflow", "wenoz", "hlld", 3, True)])
def test_chunks(n, dtype, bc, limiter, riemann, order, glm):
    assert_several_planes(*stage_march(n, dtype, limiter), 4)
    check(W.make_setup("march", 3, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, limiter=limiter, bc=((bc, bc),) * 3,
                       time_order=order, glm=glm), waves(n), dtype)


@pytest.mark.parametrize("n", [(67, 4098), (700, 745)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc,limiter,riemann,order", [("periodic", "minmod", "hlld", 2), ("outflow", "mc", "hll", 3),
                                                      ("outflow", "wenoz", "hlld", 3)])
def test_strips(n, dtype, bc, limiter, riemann, order):
    assert_several_planes(*stage_march(n, dtype, limiter), 3)
    check(W.make_setup("march", 2, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, limiter=limiter, bc=((bc, bc),) * 3,
                       time_order=order), waves(n), dtype)


# 3 and 16 cells along x: the narrow tiles of the update; 17 and 67: the wide ones
@pytest.mark.parametrize("n", [(3, 515, 61), (16, 257, 131), (17, 130, 61), (67, 65, 57)],
                         ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("emf", ["mean", "upwind"])
@pytest.mark.parametrize("limiter,order", [("mc", 2), ("wenoz", 3)])
def test_constrained_transport(n, dtype, emf, limiter, order):
    width = 16 if n[0] <= 16 else 64
    assert_several_planes(*stage_march(n, dtype, limiter), 4)
    assert_several_planes(n[2], march(*n, 512 // width, 2, 1.0, width), 3)
    if emf == "upwind":
        assert_several_planes(n[2], march(*n, 8, 2 if dtype == "f32" else 1, 2.0), 4)
    setup, V = W.cpa_wave_3d_ct(n, limiter=limiter, time_order=order, emf=emf)
    o, Ug, Uo = check(setup, V, dtype)
    scale = np.abs(Uo[9:]).max()
    for q in (9, 10, 11):
        assert np.abs(Ug[q] - Uo[q]).sum() <= TOL[dtype] * np.abs(Uo[9:]).sum()
        assert np.abs(Ug[q] - Uo[q]).max() <= TOL_MAX[dtype] * scale
    div = np.abs(face_divergence(Ug, o.dx)).max() * min(o.dx) / scale
    assert div <= (1e-13 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("bc,limiter,riemann", [("periodic", "minmod", "hlld"), ("outflow", "mc", "hll")])
def test_adjoint(bc, limiter, riemann):
    """FP64, whose limiters switch where the reference's do, against the
    reference gradient."""
    import torch

    from oracle import torch_ref as R
    from paper_2510_24175_amd.mhd import Context

    n = (3, 515, 61)
    assert_several_planes(n[2], march(*n, 4, 1, 1.2), 4)
    setup = W.make_setup("march", 3, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, limiter=limiter, bc=((bc, bc),) * 3)
    rng = np.random.default_rng(7)
    V = waves(n)
    V += 0.01 * rng.normal(size=V.shape)  # no ties
    o = C.Oracle(setup)
    U = o.prim_to_cons(V)
    dt, ch = o.cfl(U)
    damp = o.damp(dt, ch)
    lam = torch.from_numpy(rng.normal(size=U.shape))
    ctx = Context(setup, "f64", adjoint=True)
    got = ctx.step_adjoint(torch.from_numpy(U).cuda(), None, lam.cuda(), ctx.empty(), dt, ch, damp).cpu()
    Ut = torch.from_numpy(U).requires_grad_(True)
    (ref,) = torch.autograd.grad((lam * R.step(Ut, setup, dt, ch, damp)).sum(), Ut)
    assert ((got - ref).norm() / ref.norm()).item() <= 1e-10
    ctx.close()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("limiter,riemann", [("minmod", "hlld"), ("mc", "hll")])
def test_adjoint_of_a_shifted_state(dtype, limiter, riemann):
    """Periodic along z: the adjoint of the state and cotangent shifted by some
    planes, which puts every cell elsewhere in its chunk, is the shifted adjoint
    bit for bit (a chunk's first planes are formed by the same loop)."""
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = (67, 65, 58)
    assert_several_planes(n[2], march(*n, 8 if dtype == "f32" else 4, 1, 1.2), 4)
    setup = W.make_setup("march", 3, n, gamma=5.0 / 3.0, cfl=0.3, riemann=riemann, limiter=limiter)
    ctx = Context(setup, dtype, adjoint=True)
    U = ctx.prim_to_cons(torch.from_numpy(waves(n)).cuda())
    dt, ch = ctx.cfl_dt(U)
    damp = ctx.damp(dt, ch)
    U1 = torch.empty_like(U)
    ctx.step(U, torch.empty_like(U), dt, ch, damp, U1_out=U1)
    lam = torch.randn(U.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    want = ctx.step_adjoint(U, U1, lam, torch.empty_like(lam), dt, ch, damp)
    for shift in (1, 2, 5, 31):
        roll = lambda x: torch.roll(x, shift, 1).contiguous()
        got = ctx.step_adjoint(roll(U), roll(U1), roll(lam), torch.empty_like(lam), dt, ch, damp)
        assert torch.equal(got, roll(want)), shift
    ctx.close()
