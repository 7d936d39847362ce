"""GPU parity of the recycled warm start of Step 1 (ope_set_recycle): the
inner CG solves for the correction d = Y - U Lam^{-1}, starting from the
previous step's converged correction.

* Steps with the CG capped at k iterations (plain CG and the multigrid-
  preconditioned CG) equal the oracle's steps whose textbook CG starts from
  Y0 = U Lam^{-1} + d_prev, d_prev = Y_prev - U_prev Lam_prev^{-1} (the first
  step from U Lam^{-1}), to 1e-11 relative after three steps.
* A solve with recycling reaches the dense eigenvalues (1e-10) with fewer
  inner iterations than without it (a tenth fewer with plain CG, a third
  fewer with the preconditioner).
* Mixed-precision contexts and the problems of a batch are refused.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_common import say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _op(p):
    return O.Operator(p.grid.m, p.grid.h, p.V, kinetic=p.kinetic, shift=p.shift)


@pytest.mark.parametrize("mg", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_capped_recycled_steps_equal_oracle(k, mg):
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=13, N=6, seed=21)
    op = _op(p)
    tau = 20.0
    steps = 3
    say(f"recycled steps k={k} mg={mg}")
    with ope.Context(p.grid, p.V, p.N) as c:
        if mg:
            ope.ope_set_multigrid(c.handle, True)
        ope.ope_set_inner(c.handle, 0.0, 1e-30, k)           # exactly k CG iterations per step
        ope.ope_set_recycle(c.handle, True)
        Ud = to_dev(p.U0)
        its = [ope.ope_step(c.handle, Ud, tau).inner_iterations for _ in range(steps)]
        U_gpu = to_host(Ud)
    pre = O.Hierarchy(op).vcycle if mg else None
    U = p.U0.copy()
    D = np.zeros_like(U)
    for _ in range(steps):
        Li = np.linalg.inv(U.T @ O.apply_H(op, U))
        Y0 = U @ Li + D
        if mg:
            Y = O.pcg_source(op, U, Y0=Y0, tol=1e-30, max_iter=k, precond=pre)
        else:
            Y = O.cg_source(op, U, Y0=Y0, tol=1e-30, max_iter=k)
        D = Y - U @ Li
        U = O.step_general(U, Y, tau)["U"]
    assert its == [k] * steps
    assert np.max(np.abs(U_gpu - U)) <= 1e-11 * np.max(np.abs(U))


@pytest.mark.parametrize("mg", [False, True])
def test_recycled_solve_reaches_dense_eigenvalues(mg):
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=12, N=7, seed=22)          # lambda_7 = 85.5, lambda_8 = 100.8: a closed level shell
    tau = 20.0
    lam = np.linalg.eigvalsh(O.assemble_H(_op(p)).toarray())[:p.N]
    out = {}
    for rec in (False, True):
        say(f"recycled solve mg={mg} recycle={rec}")
        with ope.Context(p.grid, p.V, p.N) as c:
            if mg:
                ope.ope_set_multigrid(c.handle, True)
            if rec:
                ope.ope_set_recycle(c.handle, True)
            Ud = to_dev(p.U0)
            s = ope.ope_solve(c.handle, Ud, tau, 1e-9, 5000)
            res, ritz, drift = ope.ope_residual(c.handle, Ud, p.N)
        assert s.converged and drift <= 1e-12
        assert np.max(np.abs(np.sort(ritz) - lam) / lam) <= 1e-10
        out[rec] = s.inner_iterations
    # measured: plain CG 1554 against 1897 iterations; with the preconditioner
    # each step needs only a couple, and about half of them go
    assert out[True] < (0.7 if mg else 0.9) * out[False]


def test_recycle_refusals():
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=10, N=4, seed=23)
    with ope.Context(p.grid, p.V, p.N, precision=ope.OPE_MIXED) as c:
        with pytest.raises(ope.OpeError) as ei:
            ope.ope_set_recycle(c.handle, True)
        assert ei.value.status == ope.OPE_EUNSUPPORTED
    with ope.Batch([p]) as b:
        with pytest.raises(ope.OpeError) as ei:
            ope.ope_set_recycle(b.context(0), True)
        assert ei.value.status == ope.OPE_EUNSUPPORTED
    with ope.Context(p.grid, p.V, p.N) as c:
        ope.ope_set_recycle(c.handle, True)
        ope.ope_set_recycle(c.handle, False)
        Ud = to_dev(p.U0)
        ope.ope_step(c.handle, Ud, 10.0)                     # plain warm start again


@pytest.mark.parametrize("k", [1, 2, 3])
def test_capped_recycled_steps_by_sweeps_equal_oracle(k, monkeypatch):
    """The capped plain-CG steps on a grid of more than 16384 points, whose CG runs
    the marching sweeps."""
    real = W.wells_3d
    monkeypatch.setattr(W, "wells_3d", lambda m, N, seed: real(m=26, N=N, seed=seed))
    test_capped_recycled_steps_equal_oracle(k, False)
