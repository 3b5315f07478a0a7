"""FP64 reciprocal and square root: the IEEE results, also for the arguments
that shorter refinements of the hardware estimates round the wrong way.

With gamma = 2, no motion and no field, p = E and c^2 = 2 p / rho: a density rho
with E = 1/2 gives c_h = sqrt(1 / rho), unit density with E = x / 2 gives c_h =
sqrt(x), every other operation being exact, so c_h equals the IEEE value bit
for bit.
"""
import numpy as np
import pytest

from paper_2510_24175_amd import workloads as W

pytestmark = pytest.mark.gpu

# arguments whose reciprocal y (1 + e + e^2) is an ulp off (y the estimate, e = 1 - x y)
RECIPROCAL = ["0x1.7ff799678f7f9p-2", "0x1.fe08ac75feb1bp-2", "0x1.fefeffc118353p-2", "0x1.fca6db033ef2ep-2",
              "0x1.571b3ddcb8166p-2", "0x1.feff1f1d48b89p-2", "0x1.ffefbb12d6107p-2"]
# arguments whose root is an ulp off with one correction by the estimate's own y / 2
ROOT = ["0x1.d72520947969cp-1", "0x1.cca56d61a1ae4p-2", "0x1.2dca93a4721bp-1", "0x1.954962b7d8a9bp-2",
        "0x1.0e1b82040e84fp-1", "0x1.8de8a0c78f86ap-1", "0x1.f94c4df78409bp-2"]


def sound_speed(rho, energy):
    import torch

    from paper_2510_24175_amd.mhd import Context

    ctx = Context(W.make_setup("rest", 1, (2,), gamma=2.0, cfl=0.4, glm=False), "f64")
    U = torch.zeros(ctx.shape, dtype=torch.float64, device="cuda")
    U[0], U[4] = rho, energy
    return ctx.cfl_dt(U)[1]


@pytest.mark.parametrize("rho", RECIPROCAL)
def test_reciprocal_of_the_density(rho):
    rho = float.fromhex(rho)
    assert sound_speed(rho, 0.5) == np.sqrt(1.0 / rho)


@pytest.mark.parametrize("x", ROOT)
def test_square_root(x):
    x = float.fromhex(x)
    assert sound_speed(1.0, 0.5 * x) == np.sqrt(x)


@pytest.mark.parametrize("rho", [2.3e-308, 1.5e-308, 6e-309, 1e299])
def test_densities_at_the_ends_of_the_range(rho):
    """p = rho / 2: the speed is one, up to the rounding of 1 / rho (half an ulp),
    of its product with 2 p and of the roots."""
    assert abs(sound_speed(rho, 0.5 * rho) - 1.0) <= 4 * 2.0 ** -53
