"""GPU test of the brick kernel that steps small lattices, bitwise against the marching kernel:
lattices thinner than a brick or one cell past it in every direction, each z face rule, lateral
walls, inflow and outlet, every population storage, around the size where the smaller brick
gives way to the larger one."""
import numpy as np
import pytest

from paper_1705_03141_amd import lbm
from paper_1705_03141_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(name):
    if name.startswith("drop"):
        dims = tuple(int(k) for k in name.split()[1].split("x"))
        return W.static_droplet(dims=dims, radius=0.3 * min(dims) + 0.5, rho_r0=1.5, rho_b0=1.0, nu=0.05, A=0.01)
    if name == "box":
        pb = W.static_droplet(dims=(37, 29, 23), radius=6.0, rho_r0=1.5, rho_b0=1.0, nu=0.05, A=0.01,
                              center=(4.0, 5.5, 11.0))
        pb.faces = (W.FREESLIP,) * 6
        return pb
    if name == "rt":
        return W.rayleigh_taylor(width=17, height=45, g=1e-4, reynolds=64.0)
    return W.jet(nx=30, ny=21, nz=47, diameter=8.0, eta=4.2,
                 lateral=W.FREESLIP if name == "jet between walls" else W.PERIODIC)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("name", ["drop 1x1x1", "drop 3x1x2", "drop 8x4x4", "drop 17x5x9", "drop 32x32x32",
                                  "drop 33x32x32", "drop 50x51x51", "box", "rt", "jet", "jet between walls"])
def test_bricks_match_columns(name, storage):
    pb = _problem(name)
    assert pb.ncells <= 1 << 17, "too large for bricks: the case would not test them"
    a, b = lbm.Lattice(pb, storage=storage), lbm.Lattice(pb, storage=storage, tiling=(32, 8, 5))
    for steps in (1, 8):
        a.step(steps)
        b.step(steps)
        pa, pc = a.populations(), b.populations()
        assert np.isfinite(pa).all() and np.array_equal(pa, pc), steps
    a.close()
    b.close()
