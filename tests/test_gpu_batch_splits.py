"""Batched solves over every work split, number of right-hand sides and window
form: a wave takes entries of one right-hand side in the shift update (4, 2 or 1
waves each), finishes one in the four-thread operator, and the base shift is
updated with the window where the window is longer than one iteration."""
import numpy as np
import pytest

import synth
from oracle import dirac
from oracle.solvers import true_residuals
from paper_1710_09178_amd import stag
from tests.gpu_util import dev, host, log

pytestmark = pytest.mark.gpu

# less than a tile, remainders, and tiles in z-slab order (64-site planes)
DIMS = [(2, 2, 2, 2), (6, 4, 2, 10), (16, 8, 8, 2)]
POLES = list(np.logspace(-3, 0, 5))


@pytest.mark.parametrize("window", [1, 2, 8])
@pytest.mark.parametrize("tps", [1, 2, 4, 8])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4])
def test_batch_splits(nrhs, tps, window):
    """Stopping criterion 1e-10 on the recursive residuals; the oracle's true
    residuals may exceed it by the roundings of some 100 iterations (1e-12)."""
    log(f"batch nrhs={nrhs} tps={tps} window={window}")
    rng = synth.make_rng(510, nrhs)
    Us = [synth.random_su3_near_identity(d, 0.4, rng) for d in DIMS]
    masses = list(rng.uniform(0.02, 0.05, len(DIMS)))
    bs = [[synth.gaussian_half_vector(d, rng) for _ in range(nrhs)] for d in DIMS]
    B = stag.Batch(DIMS, nrhs)
    for i, U in enumerate(Us):
        B.set_gauge(i, dev(U))
    B.set_tps(tps)
    B.set_shift_window(window)
    rat = {"c0": 0.0, "pole": POLES, "residue": [1.0] * len(POLES)}
    packed = np.concatenate([b.reshape(-1) for per in bs for b in per])
    x = host(B.solve(masses, rat, dev(packed), tol=1e-10)[0])
    off = 0
    for d, U, m, per in zip(DIMS, Us, masses, bs):
        vh = d[0] * d[1] * d[2] * d[3] // 2
        A = lambda v: dirac.apply_A(U, v, d, m)
        for b in per:
            xs = [x[k, off:off + 3 * vh].reshape(vh, 3) for k in range(len(POLES))]
            off += 3 * vh
            assert true_residuals(A, b, POLES, xs).max() < 1.02e-10
