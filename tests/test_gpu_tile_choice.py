"""GPU test of the tile shapes that are chosen when none is set: 64 x 4 unless 32 x 8 saves enough
work, by lattice and storage, and one shape for the small lattices of a batch."""
import numpy as np
import pytest

from paper_1705_03141_amd import lbm
from paper_1705_03141_amd import workloads as W

pytestmark = pytest.mark.gpu


def _drop(*dims):
    return W.static_droplet(dims=dims, radius=0.2 * min(dims), rho_r0=1.5, rho_b0=1.0, nu=0.05, A=0.01)


@pytest.mark.parametrize("dims,storage,want", [
    ((70, 70, 70), "f32", (32, 8)),       # saves a seventh
    ((200, 100, 64), "f32", (64, 4)),    # the same work
    ((330, 100, 100), "f32", (64, 4)),    # saves a twentieth
    ((60, 60, 60), "f32", (64, 4)), ((60, 60, 60), "bf16", (32, 8)),  # the same work
])
def test_single(dims, storage, want):
    lat = lbm.Lattice(_drop(*dims), storage=storage)
    lat.step(2)
    assert lat.tiling()[:2] == want
    other = lbm.Lattice(_drop(*dims), storage=storage, tiling=(32, 4, 0))
    other.step(2)
    assert np.array_equal(lat.field("rho_r"), other.field("rho_r"))
    lat.close()
    other.close()


@pytest.mark.parametrize("sizes,storage,want", [
    ((30, 40, 50, 62), "f32", {(32, 8)}), ((40, 56, 64), "f32", {(64, 4)}), ((40, 56, 64), "bf16", {(32, 8)}),
    ((96, 112), "f16", {(32, 8), (64, 4)})])
def test_batch(sizes, storage, want):
    b = lbm.Batch([_drop(n, n, 24) for n in sizes], storage=storage)
    b.step(1)
    b.sync()
    assert {c.tiling()[:2] for c in b.cases} == want
    b.close()


@pytest.mark.parametrize("dims", [(256, 256, 2), (360, 360, 1), (256, 2, 256), (150, 150, 5)])
def test_flat_lattices_are_not_stepped_by_bricks(dims):
    """Bricks of four planes, half empty there, take 1.2 to 1.6 times as long as columns."""
    times = {}
    lats = {t: lbm.Lattice(_drop(*dims), tiling=t) for t in (None, (64, 4, 0), (32, 8, 0))}
    for _ in range(4):
        for t, lat in lats.items():
            lat.step(50)
            lat.sync()
            times.setdefault(t, []).append(lat.last_step_kernel_ms())
    pops = {t: lat.populations() for t, lat in lats.items()}
    for lat in lats.values():
        lat.close()
    assert np.array_equal(pops[None], pops[(64, 4, 0)]) and np.array_equal(pops[None], pops[(32, 8, 0)])
    assert min(times[None]) < 1.12 * min(min(times[(64, 4, 0)]), min(times[(32, 8, 0)]))
