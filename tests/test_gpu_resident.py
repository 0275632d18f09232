"""GPU tests of the one-launch (resident) multi-shift CG: against the launch
loops over the grids it takes, the way back to them when a wait inside it is
given up, and solves of several handles at once."""
import threading

import numpy as np
import pytest
import torch

import synth
from oracle import dirac
from oracle.solvers import true_residuals
from paper_1710_09178_amd.stag import LINKS_F64_12, Lattice
from tests.gpu_util import dev, host, lattice, log

pytestmark = pytest.mark.gpu


def _problem(dims, seed, eps=0.3):
    rng = synth.make_rng(0, seed)
    return synth.random_su3_near_identity(dims, eps, rng), synth.gaussian_half_vector(dims, rng)


def _solve(lat, mass, rat, tol, bd, **kw):
    xs = [lat.new_vec() for _ in rat["pole"]]
    info = lat.multishift_solve(mass, rat, tol, 100000, bd, xs, None, true_resid=False, **kw)
    return np.stack([host(x) for x in xs]), info


# 8 sites (one part of a tile), 2 tiles, 15 (ragged), 33 (the first grid that
# adds its sums by groups), 45 (ragged groups), 237 (ragged everything), 256 (a
# tile per CU)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 4), (8, 6, 4, 10), (4, 6, 8, 22), (6, 10, 8, 12),
                                  (18, 14, 10, 12), (16, 16, 16, 8)])
@pytest.mark.parametrize("links12", [False, True])
def test_matches_launch_loop(dims, links12):
    """Both loops run the same recurrences to the same stop: iteration counts
    within one, solutions within 2 tol kappa_k (both residuals are below tol)."""
    log(f"resident vs launch loop dims={dims} links12={links12}")
    U, b = _problem(dims, 31)
    rat = synth.load_rational("xm050_n12_m0.02")
    mass, tol = 0.02, 1e-11
    lat = lattice(dims, U)
    if links12:
        lat.set_link_format(LINKS_F64_12)
    bd = lat.vec_import(dev(b), 0)
    x, info = _solve(lat, mass, rat, tol, bd)
    lat.set_fused_iteration(2)
    y, infoy = _solve(lat, mass, rat, tol, bd)
    assert abs(info["iters"] - infoy["iters"]) <= 1
    for k, s in enumerate(rat["pole"]):
        kappa = (4 * mass * mass + 64 + s) / (4 * mass * mass + s)
        assert np.linalg.norm(x[k] - y[k]) <= 2 * tol * kappa * np.linalg.norm(y[k])


def test_given_up_wait_falls_back(monkeypatch):
    """With no patience every wait that misses its first poll is given up: the
    solve is then the launch loop's, bit for bit, and stays there."""
    dims = (8, 6, 4, 10)
    U, b = _problem(dims, 32)
    rat = synth.load_rational("xm050_n12_m0.02")
    ref = lattice(dims, U)
    ref.set_fused_iteration(2)
    y, infoy = _solve(ref, 0.02, rat, 1e-10, ref.vec_import(dev(b), 0))
    monkeypatch.setenv("STAG_RESIDENT_WAIT_US", "0")
    lat = Lattice(dims)
    monkeypatch.delenv("STAG_RESIDENT_WAIT_US")
    lat.set_gauge(dev(U))
    bd = lat.vec_import(dev(b), 0)
    for _ in range(2):
        x, info = _solve(lat, 0.02, rat, 1e-10, bd)
        assert info["iters"] == infoy["iters"] and np.array_equal(x, y)
    # the refinement of the precision form, too
    xs = [lat.new_vec() for _ in rat["pole"]]
    chk = lat.multishift_solve_mixed(0.02, rat, 1e-10, 100000, bd, xs, None)
    assert max(chk["true_resid"]) < 1e-10


@pytest.mark.parametrize("sloppy", [2, 3])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (18, 14, 10, 12)])
def test_mixed_refinement(dims, sloppy):
    """The refinement in resident chunks: every pole's true residual (the
    oracle's operator) below tol."""
    U, b = _problem(dims, 33, 0.2)
    rat = synth.load_rational("xm050_n12_m0.02")
    lat = lattice(dims, U)
    xs = [lat.new_vec() for _ in rat["pole"]]
    lat.multishift_solve_mixed(0.02, rat, 1e-10, 100000, lat.vec_import(dev(b), 0), xs, None, sloppy=sloppy)
    got = [host(lat.vec_export(x, 0)) for x in xs]
    res = true_residuals(lambda v: dirac.apply_A(U, v, dims, 0.02), b, rat["pole"], got)
    assert max(res) < 1e-10, res


def test_handles_on_several_threads():
    """Three handles solving at the same time on three threads and streams give
    what each gives alone, bit for bit."""
    rat = synth.load_rational("xm050_n12_m0.02")
    work = []
    for i, dims in enumerate([(16, 16, 16, 8), (8, 8, 8, 8), (18, 14, 10, 12)]):
        U, b = _problem(dims, 40 + i)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            lat = Lattice(dims)
            lat.set_gauge(dev(U))
            bd = lat.vec_import(dev(b), 0)
            xs = [lat.new_vec() for _ in rat["pole"]]
        work.append((lat, bd, xs, stream))
    torch.cuda.synchronize()

    def solve(w, out):
        lat, bd, xs, stream = w
        with torch.cuda.stream(stream):
            lat.multishift_solve(0.02, rat, 1e-10, 100000, bd, xs, None, true_resid=False)
        stream.synchronize()
        out.append(torch.stack(xs).cpu())

    alone = []
    for w in work:
        out = []
        solve(w, out)
        alone.append(out[0])
    outs = [[] for _ in work]

    def many(w, out):
        for _ in range(4):
            solve(w, out)

    threads = [threading.Thread(target=many, args=(w, o)) for w, o in zip(work, outs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for o, ref in zip(outs, alone):
        assert len(o) == 4 and all(torch.equal(x, ref) for x in o)
