"""The gauge force and the plaquette at the edges of their tiles (64 and 128
sites of one parity): less than a tile, a whole number of tiles, a remainder,
one tile past a whole round of the eight XCDs, and the z-slab order of tiles."""
import numpy as np
import pytest

import synth
from oracle import gauge
from tests.gpu_util import dev, host, lattice, log, rel_err

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (4, 4, 4, 4), (6, 2, 10, 2), (6, 6, 6, 10), (16, 8, 8, 2), (16, 16, 8, 2)]


@pytest.mark.parametrize("dims", DIMS)
def test_gauge_force_and_plaquette_tiles(dims):
    """A force component is a sum of 6 loops of 4 links: some 100 roundings of
    terms of order one, so 1e-13 of the force's norm; the mean plaquette and
    the kick round less."""
    log(f"gauge tiles dims={dims}")
    rng = synth.make_rng(210, 0)
    U = synth.random_su3_near_identity(dims, 0.6, rng)
    lat = lattice(dims, U)
    mom = lat.new_mom()
    lat.gauge_force(5.4, mom, 0.0)
    exp = gauge.gauge_force(U, dims, 5.4)
    assert rel_err(host(lat.mom_export(mom)), exp) < 1e-13
    P = synth.gaussian_momentum(dims, rng)
    m2 = lat.mom_import(dev(P))
    lat.gauge_force(5.4, m2, 0.05)
    assert rel_err(host(lat.mom_export(m2)), P + 0.05 * exp) < 1e-13
    S, plaq = lat.gauge_action(5.4)
    assert np.isclose(plaq, gauge.mean_plaquette(U, dims), rtol=0, atol=1e-13)
    assert np.isclose(S, gauge.gauge_action(U, dims, 5.4), rtol=1e-11, atol=0)
