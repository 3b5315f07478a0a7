"""WENO-Z on states in units far from one.  The equations and the scheme
scale: density, pressure and energy times 4^m and the field times 2^m give the
same velocities and the scaled state, and every rounding scales with them,
except for eps (1e-40 in FP64, 1e-30 in FP32) beside the smoothness indicators,
which here are above 1e-15 where they are not exactly zero: a change of a
weight below its rounding.  So the scaled step equals the plain one up to a
few ulps of each component.

The scales put the neighbouring cells' differences at 2e18 (FP32) and 4e25
(FP64): the indicators fit, four times as large they still do, but the sum of
three of those (FP32) or its product over both faces (FP64) does not.
"""
import numpy as np
import pytest

from paper_2510_24175_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("riemann", ["hll", "hlld"])
@pytest.mark.parametrize("dtype,m,amp", [("f32", 31, 1.0), ("f64", 43, 0.8), ("f32", -10, 1.0),
                                         ("f64", -10, 1.0)])
def test_scaled_state(dtype, m, amp, riemann):
    import torch

    from paper_2510_24175_amd.mhd import Context

    n = 67
    setup = W.make_setup("scaled", 1, (n,), gamma=5.0 / 3.0, cfl=0.4, riemann=riemann, limiter="wenoz", time_order=3,
                         glm=False)
    x = 2 * np.pi * (np.arange(n) + 0.5) / n
    V = np.zeros((9, 1, 1, n))
    # eight to nine cells a wavelength: no candidate is smooth
    V[0, 0, 0] = 1.0 + amp * (0.4 * np.sin(8 * x) + 0.2 * np.sin(7 * x + 1.0))
    V[1, 0, 0] = 0.3 * np.sin(8 * x + 0.5)
    V[2, 0, 0] = 0.2 * np.cos(7 * x)
    V[4, 0, 0] = 1.0 + amp * (0.4 * np.cos(8 * x) + 0.2 * np.sin(9 * x))
    V[5] = 0.5
    V[6, 0, 0] = 0.4 * np.sin(8 * x + 0.3)
    ctx = Context(setup, dtype)
    U = ctx.prim_to_cons(torch.from_numpy(V).cuda())
    scale = torch.tensor([4.0 ** m] * 5 + [2.0 ** m] * 3 + [1.0], dtype=U.dtype, device="cuda").reshape(9, 1, 1, 1)
    dt, ch = ctx.cfl_dt(U)
    dts, chs = ctx.cfl_dt(U * scale)
    eps = 2.0 ** -52 if dtype == "f64" else 2.0 ** -23
    assert abs(dts / dt - 1) <= 4 * 2.0 ** -52 and abs(chs / ch - 1) <= 4 * 2.0 ** -52
    plain, scaled = torch.empty_like(U), torch.empty_like(U)
    ctx.step(U, plain, dt, ch)
    ctx.step(U * scale, scaled, dt, ch)
    ctx.step_info()  # raises where a cell is not physical
    err = (scaled / scale - plain).double().abs().amax(dim=(1, 2, 3))
    err /= plain.double().abs().amax(dim=(1, 2, 3)).clamp_min(1e-30)
    print(dtype, m, riemann, [f"{e:.1e}" for e in err.tolist()], flush=True)
    assert (err[:8] <= 8 * eps).all()
