"""The caller's stream and the calls of a model: what the caller's own kernels
wrote before a call is read by it, what it writes is there for the kernels that
follow; operators recorded into a graph after such a call, and after one that
failed, replay."""
import pytest
import torch

import synth
from paper_1710_09178_amd import stag
from tests.gpu_util import dev, log

pytestmark = pytest.mark.gpu


def _lattice(dims, stream, seed):
    rng = synth.make_rng(540, seed)
    lat = stag.Lattice(dims, stream=stream)
    lat.set_gauge(dev(synth.random_su3_near_identity(dims, 0.3, rng)))
    return lat, lat.vec_import(dev(synth.gaussian_half_vector(dims, rng)), 0)


@pytest.mark.parametrize("side", [False, True])
def test_model_calls_follow_the_callers_kernels(side):
    """Targets and momenta written by the caller's kernels, behind a queue of
    products, and momenta read by them right after: the same bits as with a
    device synchronisation around every call."""
    log(f"model calls between the caller's kernels side={side}")
    dims = (16, 16, 16, 8)
    stream = torch.cuda.Stream() if side else torch.cuda.default_stream()
    with torch.cuda.stream(stream):
        lat, _ = _lattice(dims, stream, 0)
        T, M = lat.new_mom(), lat.random_momentum(3, 1)
        lat.gauge_force(5.4, T, 0.0)
        slow = torch.rand(4096, 4096, device="cuda")
        torch.cuda.synchronize()

        def run(sync):
            def wait():
                if sync:
                    torch.cuda.synchronize()
                else:
                    for _ in range(4):
                        slow @ slow

            sur = stag.Surrogate(lat, 1, seed=5)
            target, mom = torch.zeros_like(T), torch.zeros_like(T)
            out = []
            torch.cuda.synchronize()
            wait()
            target.copy_(T)
            out.append(torch.tensor(sur.eval(target)[0]))
            target.zero_()
            torch.cuda.synchronize()
            wait()
            target.copy_(T)
            sur.add_pair(target)
            target.zero_()
            out.append(torch.tensor(sur.train(2, 1e-3)))
            wait()
            mom.fill_(1.0)
            sur.force(mom, 0.0)
            out.append(mom.clone())
            torch.cuda.synchronize()
            wait()
            mom.copy_(M)
            sur.force(mom, 0.5)
            mom.mul_(2.0)
            torch.cuda.synchronize()
            return out + [mom]

        for got, ref in zip(run(False), run(True)):
            assert torch.equal(got, ref)


@pytest.mark.parametrize("side", [False, True])
def test_parameters_change_between_the_kernels_that_read_them(side):
    """Parameters set right after a force are the next force's, and the array
    they came from is free again when the call returns."""
    log(f"parameters set behind a force side={side}")
    dims = (16, 16, 16, 8)
    stream = torch.cuda.Stream() if side else torch.cuda.default_stream()
    with torch.cuda.stream(stream):
        lat, _ = _lattice(dims, stream, 3)
        sur, mom, slow = stag.Surrogate(lat, 1, seed=5), lat.new_mom(), torch.rand(4096, 4096, device="cuda")
        params = [sur.get_params(), stag.Surrogate(lat, 1, seed=6).get_params()]

        def forces(sync):
            out = []
            for k in range(6):
                p = params[k % 2].copy()
                sur.set_params(p)
                p[:] = float("nan")
                if sync:
                    torch.cuda.synchronize()
                elif k % 3 == 2:
                    slow @ slow
                sur.force(mom, 0.0)
                out.append(mom.clone())
                if sync:
                    torch.cuda.synchronize()
            assert (sur.get_params() == params[1]).all()
            return out

        ref = forces(True)
        assert not torch.equal(ref[0], ref[1])
        for got, exp in zip(forces(False), ref):
            assert torch.equal(got, exp)


def _captured_operator_replays(lat, src, stream):
    a, out, ref = lat.new_vec(), lat.new_vec(), lat.new_vec()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lat.mdagm(out, a, 0.1)
    for k in range(3):
        a.copy_((k + 1) * src)
        graph.replay()
        lat.mdagm(ref, a, 0.1)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_capture_after_model_calls_and_failures():
    log("capture after a model call and after a failed trajectory")
    dims = (8, 6, 4, 10)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lat, src = _lattice(dims, stream, 1)
        lat.mdagm(lat.new_vec(), src, 0.1)
        sur, mom = stag.Surrogate(lat, 1, seed=5), lat.new_mom()
        sur.force(mom, 0.0)
        _captured_operator_replays(lat, src, stream)
        r = [synth.load_rational(t) for t in ("xm050_n12_m0.02", "xm050_n20_m0.02", "xp025_n20_m0.02")]
        with pytest.raises(stag.StagError) as err:
            lat.trajectory(5.4, 0.02, 0.1, 2, *r, maxiter=1)
        assert err.value.code == stag.STAG_ERR_NOT_CONVERGED and "maxiter" in str(err.value)
        _captured_operator_replays(lat, src, stream)


@pytest.mark.parametrize("fmt,naik", [(stag.LINKS_F64_12, False), (stag.LINKS_F64_18, True), (stag.LINKS_F64_12, True)])
def test_operator_beside_a_graph_that_has_not_run(fmt, naik):
    """The derived links of an operator recorded into a graph are made when the
    graph runs; the same operator called before that makes its own."""
    log(f"operator beside a recorded one fmt={fmt} naik={naik}")
    dims = (8, 6, 4, 10)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lats = []
        for _ in range(2):
            lat, src = _lattice(dims, stream, 4)
            if naik:
                lat.set_naik()
            lat.set_link_format(fmt)
            lats.append(lat)
        ref, out, rec = (lats[0].new_vec() for _ in range(3))
        for k in range(2):
            lats[0].mdagm(ref, src, 0.1)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                lats[1].mdagm(rec, src, 0.1)
            lats[1].mdagm(out, src, 0.1)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref) and torch.equal(rec, ref)
            mom = lats[0].random_momentum(11, k)
            for lat in lats:
                lat.link_update(mom, 0.2)


def test_model_force_is_captured_with_the_callers_work():
    log("captured model force")
    dims = (8, 6, 4, 10)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lat, _ = _lattice(dims, stream, 2)
        sur, mom = stag.Surrogate(lat, 1, seed=5), lat.new_mom()
        ref = lat.new_mom()
        graph = torch.cuda.CUDAGraph()
        sur.force(mom, 0.0)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            sur.force(mom, 0.0)
            mom.mul_(2.0)
        for k in range(3):
            lat.link_update(lat.random_momentum(9, k), 0.1)
            graph.replay()
            sur.force(ref, 0.0)
            torch.cuda.synchronize()
            assert torch.equal(mom, 2.0 * ref)
