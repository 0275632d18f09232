"""Which loop solves what (stag_solve_loops), and that the loops agree: the
one-launch solver where it fits, the fused and the three-launch loop elsewhere
and on request, with their graphs, stops and estimates on the one-hop operator."""
import math

import numpy as np
import pytest
import torch

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


# The launch loops on the one-hop operator, which the one-launch solver replaces
# in the default mode on lattices of these sizes
def test_graph_replay_matches_direct_launches_by_mode():
    """Chunks replayed from captured graphs (captured, replayed, a second
    function's graph between them) and launched one by one: the same bits, in
    both launch loops, FP64 and FP32."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 52)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    rats = [_rat(), _rat(np.logspace(-3, 1, 6))]
    for mode in (0, 2):
        lat.set_fused_iteration(mode)
        ref = None
        for graphs in (False, True):
            lat.set_graphs(graphs)
            got = []
            for rep in range(2):
                for rat in rats:
                    x, info = _solve(lat, 0.05, rat, 1e-10, bd)
                    assert lat.solve_loops()[0] == LOOP[mode]
                    got.append((x, info["iters"]))
                xs = [lat.new_vec() for _ in POLES]
                info = lat.multishift_solve_mixed(0.05, rats[0], 1e-8, 100000, bd, xs, None)
                assert lat.solve_loops() == (LOOP[mode], "three-launch")
                got.append((np.stack([host(x) for x in xs]), info["iters"]))
            ref = ref or got
            for (x, n), (y, m) in zip(got, ref):
                assert n == m and np.array_equal(x, y)
            # solves of a kind seen before schedule their chunks from its count: the same bits
            for (x, n), (y, m) in zip(got[:3], got[3:]):
                assert n == m and np.array_equal(x, y)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("dims", [(8, 6, 4, 10), (16, 16, 16, 8)])
def test_loops_reach_the_true_residual(dims, mode):
    """Every loop's solutions by the oracle's operator; counts of iterations
    within one of the three-launch loop's."""
    log(f"loop {LOOP[mode]} dims={dims}")
    U, b = _problem(dims, 53, 0.3)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    rat = synth.load_rational("xm050_n12_m0.02")
    lat.set_fused_iteration(0)
    _, ref = _solve(lat, 0.02, rat, 1e-10, bd)
    lat.set_fused_iteration(mode)
    xs = [lat.new_vec() for _ in rat["pole"]]
    info = lat.multishift_solve(0.02, rat, 1e-10, 100000, bd, xs, None)
    assert lat.solve_loops()[0] == LOOP[mode]
    assert abs(info["iters"] - ref["iters"]) <= 1
    assert all(abs(a - c) <= 1 for a, c in zip(info["iters_per_pole"], ref["iters_per_pole"]))
    got = [host(lat.vec_export(x, 0)) for x in xs]
    res = true_residuals(lambda v: dirac.apply_A(U, v, dims, 0.02), b, rat["pole"], got)
    assert max(res) < 1e-10, res
    assert np.allclose(info["true_resid"], res, rtol=1e-3, atol=1e-15)


@pytest.mark.parametrize("sloppy", [2, 3])
def test_fp32_loops_agree(sloppy):
    """The FP32 multi-shift of each loop, refined: within 2 tol kappa_k of the
    three-launch loop's."""
    dims, mass, tol = (8, 6, 4, 10), 0.05, 1e-10
    U, b = _problem(dims, 54)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    got = {}
    for mode in (0, 1, 2):
        lat.set_fused_iteration(mode)
        xs = [lat.new_vec() for _ in POLES]
        info = lat.multishift_solve_mixed(mass, _rat(), tol, 100000, bd, xs, None, sloppy=sloppy)
        assert lat.solve_loops()[0] == LOOP[mode] and max(info["true_resid"]) < tol
        got[mode] = [host(lat.vec_export(x, 0)) for x in xs]
    for mode in (1, 2):
        for x, y, s in zip(got[mode], got[0], POLES):
            kappa = (4 * mass * mass + 64 + s) / (4 * mass * mass + s)
            assert np.linalg.norm(x - y) <= 2 * tol * kappa * np.linalg.norm(y)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("maxiter", [1, 5, 8, 9, 13, 16, 17])
def test_stop_inside_a_window_by_mode(maxiter, mode):
    """Stopped at maxiter in every position of the 8-iteration window: the
    three-launch loop's solutions at the same iteration, to rounding."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 55)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    got = {}
    for m in (0, mode):
        lat.set_fused_iteration(m)
        x, info = _solve(lat, 0.05, _rat(), 1e-10, bd, maxiter, allow_not_converged=True)
        assert info["iters"] == maxiter and lat.solve_loops()[0] == LOOP[m]
        got[m] = x
    assert np.abs(got[mode] - got[0]).max() <= 1e-12 * np.abs(got[0]).max()


@pytest.mark.parametrize("mode,lags", [(0, range(1, 9)), (1, range(2, 9)), (2, range(2, 9))])
def test_window_lengths_by_mode(mode, lags):
    """Within a loop the solutions do not depend on the window."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 56)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    lat.set_fused_iteration(mode)
    ref = None
    for lag in lags:
        lat.set_shift_window(lag)
        x, info = _solve(lat, 0.05, _rat(), 1e-10, bd)
        assert lat.solve_loops()[0] == LOOP[mode]
        ref = ref or (x, info["iters"], info["iters_per_pole"])
        assert info["iters"] == ref[1] and info["iters_per_pole"] == ref[2]
        assert np.array_equal(x, ref[0]), lag


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("mode", [0, 2])
def test_estimate_left_by_a_short_solve(mode, graphs):
    """A solve that needs more iterations than the estimate left by one of its
    kind stopped at maxiter still runs to its own stop."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 57)
    lat = lattice(dims, U)
    bd = lat.vec_import(dev(b), 0)
    lat.set_fused_iteration(mode)
    lat.set_graphs(graphs)
    x, info = _solve(lat, 0.05, _rat(), 1e-10, bd)
    _, short = _solve(lat, 0.05, _rat(), 1e-10, bd, 10, allow_not_converged=True)
    assert short["iters"] == 10
    y, again = _solve(lat, 0.05, _rat(), 1e-10, bd)
    assert again["iters"] == info["iters"] and np.array_equal(x, y)
    assert lat.solve_loops()[0] == LOOP[mode]


@pytest.mark.parametrize("mode", [0, 2])
def test_streamed_links_by_mode(mode):
    """Links of 264 MB, beyond the Infinity Cache: plain, default and streamed
    loads give the same bits in both launch loops."""
    dims = (32, 32, 32, 14)
    log(f"streamed links {dims} mode {mode}")
    lat = Lattice(dims)
    gen = torch.Generator(device="cuda").manual_seed(58)
    rows = torch.randn(2, math.prod(dims) * 4, 3, dtype=torch.complex128, device="cuda", generator=gen)
    u = rows[0] / rows[0].norm(dim=1, keepdim=True)
    v = rows[1] - (u.conj() * rows[1]).sum(1, keepdim=True) * u
    v = v / v.norm(dim=1, keepdim=True)
    lat.set_gauge(torch.stack([u, v, torch.linalg.cross(u, v).conj()], 1).reshape(-1))
    bd = lat.vec_import(torch.randn(math.prod(dims) // 2, 3, dtype=torch.complex128, device="cuda", generator=gen), 0)
    lat.set_fused_iteration(mode)
    ref = None
    for streaming in (1, 0, 2):
        lat.set_link_streaming(streaming)
        x, info = _solve(lat, 0.1, _rat(POLES[:3]), 1e-10, bd, 12, allow_not_converged=True)
        assert info["iters"] == 12 and lat.solve_loops()[0] == LOOP[mode]
        ref = x if ref is None else ref
        assert np.array_equal(x, ref)
