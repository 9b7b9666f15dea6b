"""GPU test of 16-bit batches without lateral walls against single lattices, bitwise: the step kernel
takes other forms there than for a single lattice (registers kept or formed again, the ring of
densities interleaved or not), for either tile shape, ragged lattices and a jet with its outlet."""
import numpy as np
import pytest

from paper_1705_03141_amd import lbm
from paper_1705_03141_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f16", "bf16"])
def test_matches_single_lattices(storage):
    drop = lambda *dims: W.static_droplet(dims=dims, radius=6.0, rho_r0=1.5, rho_b0=1.0, nu=0.05,  # noqa: E731
                                          A=0.01, center=(9.0, 8.5, 7.0))
    cases = [drop(70, 21, 23), drop(128, 8, 9), drop(37, 29, 11), W.jet(nx=66, ny=34, nz=40, diameter=6.0, seed=3)]
    b = lbm.Batch(cases, storage=storage)
    b.step(12)
    b.sync()
    for k, pb in enumerate(cases):
        got = b.cases[k].populations()
        assert np.isfinite(got).all()
        for tiling in (None, (64, 4, 5), (32, 8, 0), (64, 8, 4)):
            alone = lbm.Lattice(pb, storage=storage, tiling=tiling)
            alone.step(12)
            same = bool(np.array_equal(got, alone.populations()))
            alone.close()
            assert same, f"case {k} differs from its single-lattice run with tiling {tiling}"
    b.close()
