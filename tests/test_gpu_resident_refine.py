"""Mixed-precision solves whose refinement runs in one launch per stretch of
iterations (FP32, up to two tiles per CU) or in the launch loop with polls at
the expected stop: both reach the FP64 true residual at every pole."""
import numpy as np
import pytest

import synth
from paper_1710_09178_amd import stag
from tests.gpu_util import dev, host, lattice, log

pytestmark = pytest.mark.gpu

# 15 ragged tiles, 1, 256 (a tile per CU), 258 and 512 (two per CU), 513 (the loop)
DIMS = [(8, 6, 4, 10), (2, 2, 2, 2), (16, 16, 4, 32), (16, 2, 4, 258), (16, 16, 16, 16), (16, 2, 6, 342)]


@pytest.mark.parametrize("every", [3, 50])
@pytest.mark.parametrize("sloppy", [stag.LINKS_F32_18, stag.LINKS_F16_12])
@pytest.mark.parametrize("dims", DIMS)
def test_mixed_matches_double(dims, sloppy, every):
    """The refinement stops on the FP64 residual itself: at most tol.  Two
    solutions with residuals below tol differ by 2 tol kappa at most."""
    log(f"mixed refinement dims={dims} sloppy={sloppy} every={every}")
    rng = synth.make_rng(520, 0)
    lat = lattice(dims, synth.random_su3_near_identity(dims, 0.3, rng))
    b = lat.vec_import(dev(synth.gaussian_half_vector(dims, rng)), 0)
    poles = [1e-3, 3e-2, 1.0]
    rat = {"c0": 0.0, "pole": poles, "residue": [1.0] * 3}
    mass, tol = 0.05, 1e-10
    ref = [lat.new_vec() for _ in poles]
    lat.multishift_solve(mass, rat, tol, 100000, b, ref, None, true_resid=False)
    for mode in (1, 0):
        lat.set_fused_iteration(mode)
        xs = [lat.new_vec() for _ in poles]
        info = lat.multishift_solve_mixed(mass, rat, tol, 100000, b, xs, sloppy=sloppy, reliable_every=every)
        assert max(info["true_resid"]) <= tol
        for x, y, s in zip(xs, ref, poles):
            kappa = (4 * mass * mass + 64 + s) / (4 * mass * mass + s)
            assert np.linalg.norm(host(x - y)) <= 2 * tol * kappa * np.linalg.norm(host(y))
