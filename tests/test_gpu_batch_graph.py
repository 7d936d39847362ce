"""GPU tests of the graph-captured batched step (ope_batch_capture / replay).

* Replays of the captured step equal eager batched steps bit for bit (FP64
  and mixed, shared CG launches and per-problem launches, ragged grids and
  block widths), with
  the same diagnostics, over several replays with eager batched steps of
  other buffers and a host synchronisation between them; a large problem
  (48^3, N = 128) whose column sums take more than one work-group runs its
  CG on its own stream inside the graph.
* Too few captured CG iterations: every problem reports OPE_ECG_MAXIT with
  the captured count, and the block stays orthonormal.
* Refusals: odd iteration counts, a problem with N > 128, replay before
  capture.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import say, to_host

pytestmark = pytest.mark.gpu


def _dev(a, prec):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64 if prec == 0 else np.float32)).to("cuda")


def _ragged():
    return [W.wells_3d(m=13, N=5, seed=1), W.wells_3d(m=20, N=17, seed=2), W.harmonic_2d_32(),
            W.wells_3d(m=16, N=34, seed=3), W.wells_3d(m=11, N=3, seed=4), W.wells_3d(m=28, N=48, seed=5)]


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("prec", [0, 1])
def test_replays_equal_eager_steps(prec, shared):
    import torch
    from paper_2511_06788_amd import ope
    probs = _ragged() + [W.wells_3d(m=48, N=128, seed=6)]
    tau = 0.5
    say(f"graph replays vs eager steps prec={prec} shared={shared}")
    with ope.Batch(probs, precision=prec) as b:
        b.set_shared(shared)
        Ug = [_dev(p.U0, prec) for p in probs]      # stepped by the graph
        Ue = [_dev(p.U0, prec) for p in probs]      # stepped eagerly
        Uo = [_dev(p.U0, prec) for p in probs]      # other eager work between replays
        b.capture(Ug, tau, 200)
        for k in range(4):
            ig = b.replay()
            ie = b.step(Ue, tau)
            for i in range(len(probs)):
                a, c = ig[i], ie[i]
                assert a.status == c.status == ope.OPE_OK, (k, i, a.status, c.status)
                assert (a.energy, a.residual, a.drift, a.inner_iterations) == (
                    c.energy, c.residual, c.drift, c.inner_iterations), (k, i)
                assert torch.equal(Ug[i], Ue[i]), (k, i)
            b.step(Uo, 2.0 * tau)
            torch.cuda.synchronize()
        # a replay without waiting, then the caller's stream orders the read
        b.replay(wait=False)
        b.step(Ue, tau)
        torch.cuda.synchronize()
        for i in range(len(probs)):
            assert torch.equal(Ug[i], Ue[i]), ("no-wait replay", i)
        assert all(i.inner_iterations > 0 for i in ig)


def test_too_few_iterations_report_maxit():
    from paper_2511_06788_amd import ope
    probs = _ragged()[:4]
    say("graph replay with 2 CG iterations")
    with ope.Batch(probs) as b:
        b.set_shared(True)
        Ug = [_dev(p.U0, 0) for p in probs]
        b.capture(Ug, 0.5, 2)
        for _ in range(2):
            infos = b.replay(allow_maxit=True)
            for i in infos:
                assert i.status == ope.OPE_ECG_MAXIT
                assert i.inner_iterations == 2
        for U, p in zip(Ug, probs):
            Uh = to_host(U)
            assert np.all(np.isfinite(Uh))
            assert np.linalg.norm(Uh.T @ Uh - np.eye(p.N)) <= 1e-12


def test_capture_refusals():
    from paper_2511_06788_amd import ope
    small = [W.wells_3d(m=11, N=3, seed=4), W.wells_3d(m=12, N=4, seed=5)]
    with ope.Batch(small) as b:
        with pytest.raises(ope.OpeError) as ei:
            b.replay()
        assert ei.value.status == ope.OPE_EINVAL
        with pytest.raises(ope.OpeError) as ei:
            b.capture([_dev(p.U0, 0) for p in small], 0.5, 7)
        assert ei.value.status == ope.OPE_EINVAL
    wide = [W.wells_3d(m=11, N=3, seed=4), W.wells_3d(m=12, N=130, seed=5)]
    with ope.Batch(wide) as b:
        with pytest.raises(ope.OpeError) as ei:
            b.capture([_dev(p.U0, 0) for p in wide], 0.5, 8)
        assert ei.value.status == ope.OPE_EUNSUPPORTED


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("prec", [0, 1])
def test_replays_equal_eager_steps_past_the_one_launch_grids(prec, shared):
    """Several problems of more than 16384 points, of one class and of others, among
    them rows swept in wide chunks (two-launch column sums) and a 2D grid: with
    shared launches the sweeps of all of them are the graph's."""
    import torch
    from paper_2511_06788_amd import ope
    probs = [W.wells_3d(m=26, N=45, seed=1), W.wells_3d(m=27, N=16, seed=2), W.wells_3d(m=28, N=127, seed=3),
             W.wells_3d(m=26, N=16, seed=4), W.harmonic_2d_32(m=130), W.wells_3d(m=27, N=99, seed=5)]
    tau = 0.5
    say(f"graph replays of larger grids prec={prec} shared={shared}")
    with ope.Batch(probs, precision=prec) as b:
        b.set_shared(shared)
        Ug = [_dev(p.U0, prec) for p in probs]
        Ue = [_dev(p.U0, prec) for p in probs]
        Uo = [_dev(p.U0, prec) for p in probs]
        b.capture(Ug, tau, 300)
        for k in range(3):
            ig = b.replay()
            ie = b.step(Ue, tau)
            for i in range(len(probs)):
                a, c = ig[i], ie[i]
                assert a.status == c.status == ope.OPE_OK, (k, i, a.status, c.status)
                assert a.inner_iterations > 0
                assert (a.energy, a.residual, a.drift, a.inner_iterations) == (
                    c.energy, c.residual, c.drift, c.inner_iterations), (k, i)
                assert torch.equal(Ug[i], Ue[i]), (k, i)
            b.step(Uo, 2.0 * tau)
            torch.cuda.synchronize()
