"""Which loop solves what (stag_solve_loops), and that the loops agree: the
one-launch solver where it fits, the fused and the three-launch loop elsewhere
and on request, with their graphs, stops and estimates on the one-hop operator."""
import numpy as np
import pytest

import synth
from oracle import dirac
from oracle.solvers import true_residuals
from paper_1710_09178_amd.stag import Lattice
from tests.gpu_util import dev, host, lattice, log

pytestmark = pytest.mark.gpu

POLES = list(np.logspace(-4, 0, 8))


def _problem(dims, seed, eps=0.4):
    rng = synth.make_rng(0, seed)
    return synth.random_su3_near_identity(dims, eps, rng), synth.gaussian_half_vector(dims, rng)


def _rat(poles=POLES):
    return {"c0": 0.0, "pole": list(poles), "residue": [1.0] * len(poles)}


def _solve(lat, mass, rat, tol, bd, maxiter=100000, **kw):
    xs = [lat.new_vec() for _ in rat["pole"]]
    info = lat.multishift_solve(mass, rat, tol, maxiter, bd, xs, None, true_resid=False, **kw)
    return np.stack([host(x) for x in xs]), info


LOOP = {0: "three-launch", 1: "one-launch", 2: "fused"}


# 15 tiles; 256, a tile per CU; 264, where FP32 alone is still solved in one launch;
# 512, two tiles per CU; 520, where the forms for small grids end
@pytest.mark.parametrize("dims,fp64,fp32", [((8, 6, 4, 10), "one-launch", "one-launch"),
                                            ((16, 16, 16, 8), "one-launch", "one-launch"),
                                            ((16, 16, 6, 22), "fused", "one-launch"),
                                            ((16, 16, 16, 16), "fused", "one-launch"),
                                            ((16, 16, 26, 10), "three-launch", "three-launch")])
def test_route_by_size(dims, fp64, fp32):
    """The FP32 solve's shifted solutions are checked unrefined: at a tolerance of
    1e-3 and m = 0.25 the FP32 residuals (rounding 64 |x| 2^-24 <= 2e-5 |b|) meet
    it by themselves, so the refinement CGs stop at their first check, but for
    one whose residual falls between the two roundings of the tolerance."""
    log(f"route by size {dims}")
    U, b = _problem(dims, 50, 0.2)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    _solve(lat, 0.25, _rat(), 1e-8, bd)
    assert lat.solve_loops() == (fp64, "none")
    xs = [lat.new_vec() for _ in POLES]
    for sloppy in (2, 3):
        iters = []
        for mode in (0, 1):
            lat.set_fused_iteration(mode)
            info = lat.multishift_solve_mixed(0.25, _rat(), 1e-3, 100000, bd, xs, None, sloppy=sloppy,
                                              tol_sloppy=1e-3)
            assert max(info["true_resid"]) < 1e-3
            assert lat.solve_loops() == ((fp32 if mode else "three-launch"),
                                         ("one-launch" if mode and fp32 == "one-launch" else "three-launch"))
            if sloppy == 2:  # (FP16 links are another operator: those solutions are refined)
                assert info["iters"] <= max(info["iters_per_pole"]) + 1
            iters.append(info["iters"])
        assert abs(iters[0] - iters[1]) <= 2


def test_given_up_wait_is_reported(monkeypatch):
    """The launch loop solves after a given-up wait and says so."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 51)
    monkeypatch.setenv("STAG_RESIDENT_WAIT_US", "0")
    lat = Lattice(dims)
    monkeypatch.delenv("STAG_RESIDENT_WAIT_US")
    lat.set_gauge(dev(U))
    bd = lat.vec_import(dev(b), 0)
    for _ in range(20):  # with one more try among them, given up as well
        _solve(lat, 0.05, _rat(), 1e-6, bd)
        assert lat.solve_loops() == ("fused", "none")
