"""The rational sum r(A) b = c0 b + sum_k residue_k x_k of the mixed-precision
solve: of the same call's solutions, with and without the caller's own x."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, lattice, log, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (8, 6, 4, 10)])
def test_sum_of_the_mixed_solve(dims, mode):
    """Thirteen terms in FP64, added in the same order: a rounding each."""
    log(f"sum of the mixed solve dims={dims} mode={mode}")
    rng = synth.make_rng(0, 90)
    U = synth.random_su3_near_identity(dims, 0.3, rng)
    b = synth.gaussian_half_vector(dims, rng)
    lat = lattice(dims, U)
    lat.set_fused_iteration(mode)
    rat = synth.load_rational("xm050_n12_m0.02")
    bd = lat.vec_import(dev(b), 0)
    xs, s, s2 = [lat.new_vec() for _ in rat["pole"]], lat.new_vec(), lat.new_vec()
    info = lat.multishift_solve_mixed(0.05, rat, 1e-10, 100000, bd, xs, s)
    assert max(info["true_resid"]) < 1e-10
    x = [host(lat.vec_export(v, 0)) for v in xs]
    expect = rat["c0"] * b + sum(c * v for c, v in zip(rat["residue"], x))
    assert rel_err(host(lat.vec_export(s, 0)), expect) < 1e-14
    lat.multishift_solve_mixed(0.05, rat, 1e-10, 100000, bd, None, s2, true_resid=False)
    assert np.array_equal(host(lat.vec_export(s2, 0)), host(lat.vec_export(s, 0)))
