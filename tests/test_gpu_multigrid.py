"""GPU parity of the multigrid-preconditioned Step 1 (ope_set_multigrid)
against the oracle's V-cycle and preconditioned CG (oracle/multigrid.py).

* One V-cycle (ope_mg_vcycle) equals the oracle's ``Hierarchy.vcycle`` to
  1e-12 relative on 3D and 2D grids with odd and even sizes, a kinetic
  factor and a shift, a grid two nodes thick (levels one node thick), even
  and odd N, rows split into slices, and at 64^3 with N = 128 (columns
  compared against the oracle on eight of them); the hierarchy has the
  oracle's number of levels and coarsest size.
* The preconditioned CG capped at k = 1, 2, 3, 5, 6 iterations (eager and
  graph-replayed chunks; N = 40 and 17 at k = 3) equals the oracle's
  ``pcg_source`` iterate.
* Stand-alone Step 1 converges to the sparse direct solution in a few
  iterations; steps with a tight inner solve equal the oracle's exact Steps
  1-4; at 64^3 with N = 128 a step needs far fewer inner iterations than the
  plain CG, keeps the block orthonormal and lowers the energy.
* Batched steps of problems with the preconditioner equal their single steps.
* The preconditioner's default inner factor (0.25; 0.1 again when it is
  switched off, and the caller's factor once ope_set_inner was called).
* Mixed precision: the FP32 V-cycle equals the oracle's to FP32 rounding, and
  a mixed solve with the preconditioner followed by an FP64 one reaches the
  dense eigenvalues.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_common import empty_dev, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _op(p):
    return O.Operator(p.grid.m, p.grid.h, p.V, kinetic=p.kinetic, shift=p.shift)


def _ctx(p, N=None):
    from paper_2511_06788_amd import ope
    c = ope.Context(p.grid, p.V, p.N if N is None else N, kinetic=p.kinetic, shift=p.shift)
    ope.ope_set_multigrid(c.handle, True)
    return c


def _case(name):
    if name == "wells20_N8":
        return W.wells_3d(m=20, N=8, seed=3)
    if name == "aniso13x11x9_N7":
        g = W.Grid(m=(13, 11, 9), h=(0.07, 0.08, 0.1), lo=(0.0, 0.0, 0.0))
        V = W.harmonic_potential(g, 40.0, (0.5, 0.4, 0.45))
        return W.Problem("aniso", g, V, 7, 1.0, U0=W.initial_block(g.n, 7, 1), kinetic=0.5, shift=2.0)
    if name == "2d_33x27_N6":
        g = W.Grid(m=(33, 27), h=(1.0 / 34, 1.0 / 28), lo=(0.0, 0.0))
        V = W.harmonic_potential(g, 80.0, (0.5, 0.5))
        return W.Problem("2d", g, V, 6, 1.0, U0=W.initial_block(g.n, 6, 2))
    if name == "thin40x2x30_N6":
        # y has two nodes, one on the coarse levels: tiles one column high,
        # whose ring is longer than two columns per thread
        g = W.Grid(m=(40, 2, 30), h=(0.05, 0.05, 0.05), lo=(0.0, 0.0, 0.0))
        V = W.harmonic_potential(g, 30.0, (0.5, 0.5, 0.5))
        return W.Problem("thin", g, V, 6, 1.0, U0=W.initial_block(g.n, 6, 4))
    if name == "wells16_N40":
        return W.wells_3d(m=16, N=40, seed=6)         # rows in two slices of 10 vector pairs
    if name == "wells12_N17":
        return W.wells_3d(m=12, N=17, seed=8)         # odd N: one element per vector group
    raise KeyError(name)


VCYCLE_CASES = ["wells20_N8", "aniso13x11x9_N7", "2d_33x27_N6", "thin40x2x30_N6", "wells16_N40", "wells12_N17"]


@pytest.mark.parametrize("name", VCYCLE_CASES)
def test_vcycle_matches_oracle(name):
    from paper_2511_06788_amd import ope
    p = _case(name)
    op = _op(p)
    hier = O.Hierarchy(op)
    R = np.random.default_rng(7).standard_normal((p.grid.n, p.N))
    ref = hier.vcycle(R)
    say(f"mg vcycle {name}")
    with _ctx(p) as c:
        lv, nc = ope.ope_mg_info(c.handle)
        Z = empty_dev(p.grid.n, p.N)
        ope.ope_mg_vcycle(c.handle, to_dev(R), Z)
        got = to_host(Z)
    assert lv == len(hier.levels) and nc == hier.levels[-1].n
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_vcycle_full_size_matches_oracle_columns():
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=64, N=128, seed=0)
    op = _op(p)
    R = np.random.default_rng(5).standard_normal((p.grid.n, 128))
    cols = [0, 1, 37, 64, 90, 126, 127, 5]
    ref = O.Hierarchy(op).vcycle(R[:, cols])
    say("mg vcycle 64^3 N=128")
    with _ctx(p) as c:
        Z = empty_dev(p.grid.n, 128)
        ope.ope_mg_vcycle(c.handle, to_dev(R), Z)
        got = to_host(Z)[:, cols]
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 6])
def test_capped_pcg_equals_oracle_iterates(k, graphs):
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=13, N=6, seed=11)
    op = _op(p)
    U = W.initial_block(p.grid.n, p.N, 5)
    say(f"capped PCG k={k} graphs={graphs}")
    with _ctx(p) as c:
        ope.ope_set_graphs(c.handle, graphs)
        Yd = empty_dev(p.grid.n, p.N)
        its = ope.ope_source_solve(c.handle, to_dev(U), Yd, None, 1e-15, k, allow_maxit=True)
        Y = to_host(Yd)
    st = {}
    Y_ref = O.pcg_source(op, U, None, tol=1e-15, max_iter=k, stats=st)
    assert its == k and st["iterations"] == k
    assert np.max(np.abs(Y - Y_ref)) <= 1e-12 * np.max(np.abs(Y_ref))


@pytest.mark.parametrize("N", [40, 17])
def test_capped_pcg_equals_oracle_iterates_wide_rows(N):
    """The PCG dot products of the finest post-smoothing with rows split into
    slices (N = 40) and with odd N."""
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=13, N=N, seed=12)
    op = _op(p)
    U = W.initial_block(p.grid.n, p.N, 6)
    say(f"capped PCG N={N}")
    with _ctx(p) as c:
        Yd = empty_dev(p.grid.n, p.N)
        its = ope.ope_source_solve(c.handle, to_dev(U), Yd, None, 1e-15, 3, allow_maxit=True)
        Y = to_host(Yd)
    Y_ref = O.pcg_source(op, U, None, tol=1e-15, max_iter=3)
    assert its == 3
    assert np.max(np.abs(Y - Y_ref)) <= 1e-12 * np.max(np.abs(Y_ref))


def test_capped_pcg_with_a_stopped_slice():
    """Right-hand-side columns that are zero stop before the first iteration;
    with N = 40 the first 20 columns are a whole slice of the row, whose
    V-cycle work-groups return at once (writing zero partial sums) while the
    other slice iterates."""
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=13, N=40, seed=13)
    op = _op(p)
    U = W.initial_block(p.grid.n, p.N, 7)
    U[:, :20] = 0.0
    say("capped PCG N=40 with a stopped slice")
    with _ctx(p) as c:
        Yd = empty_dev(p.grid.n, p.N)
        its = ope.ope_source_solve(c.handle, to_dev(U), Yd, None, 1e-15, 3, allow_maxit=True)
        Y = to_host(Yd)
    Y_ref = O.pcg_source(op, U, None, tol=1e-15, max_iter=3)
    assert its == 3
    assert np.all(Y[:, :20] == 0.0)
    assert np.max(np.abs(Y - Y_ref)) <= 1e-12 * np.max(np.abs(Y_ref))


def test_source_solve_reaches_direct_solution():
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=24, N=5, seed=1)
    op = _op(p)
    ref = O.GSolver(op, "sparse")(p.U0)
    say("PCG source solve")
    with _ctx(p) as c:
        Yd = empty_dev(p.grid.n, p.N)
        its = ope.ope_source_solve(c.handle, to_dev(p.U0), Yd, None, 1e-11, 100)
        Y = to_host(Yd)
    assert its <= 20
    assert np.max(np.abs(Y - ref)) <= 1e-9 * np.max(np.abs(ref))


def test_steps_match_oracle_exact_steps():
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=14, N=12, seed=2)
    op = _op(p)
    G = O.GSolver(op, "sparse")
    tau = 30.0
    say("PCG steps vs oracle")
    with _ctx(p) as c:
        ope.ope_set_inner(c.handle, 0.0, 1e-13, 500)
        U = to_dev(p.U0)
        ref = p.U0
        for _ in range(4):
            info = ope.ope_step(c.handle, U, tau, allow_maxit=False)
            assert abs(info.energy - O.energy(op, ref)) <= 1e-12 * abs(info.energy)
            assert info.inner_iterations <= 40
            ref = O.steps_1_to_4(ref, G, tau)["U"]
        got = to_host(U)
    assert np.max(np.abs(got - ref)) <= 1e-10


def test_full_size_steps_need_few_iterations():
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=64, N=128, seed=0)
    tau = 45.0
    say("PCG steps 64^3 N=128")
    with ope.Context(p.grid, p.V, p.N) as plain, _ctx(p) as c:
        ope.ope_set_inner(c.handle, 0.1, 1e-12, 2000)        # the plain CG's default factor
        Ua, Ub = to_dev(p.U0), to_dev(p.U0)
        ia = [ope.ope_step(plain.handle, Ua, tau) for _ in range(3)]
        ib = [ope.ope_step(c.handle, Ub, tau) for _ in range(3)]
        res_a, _, drift_a = ope.ope_residual(plain.handle, Ua, p.N, want_ritz=False)
        res_b, _, drift_b = ope.ope_residual(c.handle, Ub, p.N, want_ritz=False)
    for a, b in zip(ia, ib):
        # the same input block on the first step
        assert b.inner_iterations * 3 <= a.inner_iterations
    assert ia[0].energy == ib[0].energy
    assert ib[2].energy < ib[1].energy < ib[0].energy
    assert drift_b <= 1e-12
    # both steps meet the same inner tolerance: the iterates stay close
    assert abs(res_b - res_a) <= 0.2 * res_a


def test_inner_factor_defaults():
    """Enabling the preconditioner sets the inner factor to 0.25 and disabling
    it back to 0.1, unless ope_set_inner chose one: steps equal those with the
    factor set explicitly, bit for bit."""
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=16, N=8, seed=5)
    tau = 45.0

    def run(setup):
        with ope.Context(p.grid, p.V, p.N) as c:
            setup(c.handle)
            U = to_dev(p.U0)
            info = [ope.ope_step(c.handle, U, tau) for _ in range(3)]
            return to_host(U), [(i.energy, i.inner_iterations) for i in info]

    say("inner factor defaults")
    mg = lambda h, on=True: ope.ope_set_multigrid(h, on)
    inner = lambda h, eta: ope.ope_set_inner(h, eta, 1e-12, 2000)
    a = run(lambda h: mg(h))
    b = run(lambda h: (inner(h, 0.25), mg(h)))
    assert np.array_equal(a[0], b[0]) and a[1] == b[1]
    c = run(lambda h: (inner(h, 0.1), mg(h)))                   # the caller's factor stays
    d = run(lambda h: (mg(h), inner(h, 0.1)))
    assert np.array_equal(c[0], d[0]) and c[1] == d[1]
    assert sum(x[1] for x in c[1]) > sum(x[1] for x in a[1])      # a tighter tolerance costs iterations
    e = run(lambda h: (mg(h), mg(h, False)))
    f = run(lambda h: None)
    assert np.array_equal(e[0], f[0]) and e[1] == f[1]


def test_batched_steps_with_multigrid_equal_single_steps():
    from paper_2511_06788_amd import ope
    probs = [W.wells_3d(m=13, N=5, seed=1), W.wells_3d(m=20, N=17, seed=2), W.harmonic_2d_32()]
    tau = 0.5
    say("batched PCG steps vs single")
    with ope.Batch(probs) as b:
        b.set_shared(True)
        for i in range(len(probs)):
            ope.ope_set_multigrid(b.context(i), True)
        Ub = [to_dev(p.U0) for p in probs]
        ib = [b.step(Ub, tau) for _ in range(2)]
        Ub = [to_host(U) for U in Ub]
    for i, p in enumerate(probs):
        with _ctx(p) as c:
            U = to_dev(p.U0)
            ia = [ope.ope_step(c.handle, U, tau) for _ in range(2)]
            U = to_host(U)
        assert np.array_equal(U, Ub[i]), i
        for k in range(2):
            assert (ia[k].energy, ia[k].inner_iterations) == (ib[k][i].energy, ib[k][i].inner_iterations)


def test_multigrid_refusals():
    from paper_2511_06788_amd import ope
    q = W.wells_3d(m=8, N=257, seed=0)
    with pytest.raises(ope.OpeError) as ei:                  # 257 single-element chunks per row
        ope.Context(q.grid, q.V, q.N)
    assert ei.value.status == ope.OPE_EUNSUPPORTED
    p = W.wells_3d(m=12, N=4, seed=0)
    with ope.Context(p.grid, p.V, p.N) as c:
        R = to_dev(p.U0)
        Z = empty_dev(p.grid.n, p.N)
        with pytest.raises(ope.OpeError):
            ope.ope_mg_vcycle(c.handle, R, Z)            # preconditioner off
        ope.ope_set_multigrid(c.handle, True)
        hier = O.Hierarchy(_op(p))
        assert ope.ope_mg_info(c.handle) == (len(hier.levels), hier.levels[-1].n)
        ope.ope_set_multigrid(c.handle, False)
        assert ope.ope_mg_info(c.handle) == (0, 0)


@pytest.mark.parametrize("name", VCYCLE_CASES)
def test_fp32_vcycle_matches_oracle(name):
    import torch
    from paper_2511_06788_amd import ope
    p = _case(name)
    hier = O.Hierarchy(_op(p))
    R = np.random.default_rng(8).standard_normal((p.grid.n, p.N)).astype(np.float32)
    ref = hier.vcycle(R.astype(np.float64))
    say(f"mg vcycle fp32 {name}")
    with ope.Context(p.grid, p.V, p.N, kinetic=p.kinetic, shift=p.shift, precision=ope.OPE_MIXED) as c:
        ope.ope_set_multigrid(c.handle, True)
        Z = torch.empty((p.grid.n, p.N), dtype=torch.float32, device="cuda")
        ope.ope_mg_vcycle(c.handle, torch.from_numpy(R).to("cuda"), Z)
        got = Z.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - ref)) <= 2e-6 * np.max(np.abs(ref))


def test_mixed_solve_with_multigrid_reaches_dense_eigenvalues():
    import torch
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=16, N=8, seed=1)
    op = _op(p)
    w = np.linalg.eigvalsh(O.assemble_H(op).toarray())
    tau = 0.8 * 2.0 / (1.0 / w[0] - 1.0 / w[-1])
    say("mixed + multigrid solve, then FP64 + multigrid")
    with ope.Context(p.grid, p.V, p.N, precision=ope.OPE_MIXED) as cm, _ctx(p) as cd:
        ope.ope_set_multigrid(cm.handle, True)
        U32 = torch.from_numpy(p.U0.astype(np.float32)).to("cuda")
        # the FP32 preconditioned CG floors the mixed phase near 1e-3 (the plain
        # FP32 CG near 1e-4): switch to FP64 there
        sm = ope.ope_solve(cm.handle, U32, tau, 1e-3, 5000)
        assert sm.converged == 1 and sm.inner_iterations < 8 * sm.steps
        U = torch.empty((p.grid.n, p.N), dtype=torch.float64, device="cuda")
        ope.ope_convert(cm.handle, U32, U, p.grid.n * p.N, True)
        sf = ope.ope_solve(cd.handle, U, tau, 1e-10, 20000)
        res, ritz, drift = ope.ope_residual(cd.handle, U, p.N)
    assert sf.converged == 1
    assert np.max(np.abs(ritz - w[:p.N]) / w[:p.N]) <= 1e-10
    assert drift <= 1e-12


@pytest.mark.parametrize("m,N", [((25, 25, 25), 3), ((26, 25, 25), 5), ((24, 26, 28), 2), ((4000, 1), 3), ((1, 97, 41), 4),
                                 ((6000, 2), 1), ((9, 7, 5), 212), ((5, 4, 4), 1), ((2, 2, 30), 6)])
def test_vcycle_at_the_edges_of_the_fused_coarse_end(m, N):
    """Grids whose levels meet the fused coarse end at its largest size (13^3 =
    2197 nodes stay outside, 12 x 13 x 14 = 2184 too, levels below go in), whose
    levels shrink along one axis only, or whose first coarse level is already
    the coarsest.  The set-up recovers the potential from the diagonal, V + 2 sum
    c_a, so it is off by eps 2 sum c_a and the result by up to that over the
    smallest eigenvalue of -Lap_h beside the sums' rounding."""
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid(m)
    rng = np.random.default_rng(len(m) * 100 + N)
    V = rng.uniform(0.0, 40.0, g.n)
    N = min(N, g.n)
    hier = O.Hierarchy(O.Operator(g.m, g.h, V))
    R = rng.standard_normal((g.n, N))
    ref = hier.vcycle(R)
    say(f"mg vcycle coarse end m={m} N={N}")
    with ope.Context(g, V, N) as c:
        ope.ope_set_multigrid(c.handle, True)
        Z = empty_dev(g.n, N)
        ope.ope_mg_vcycle(c.handle, to_dev(R), Z)
        got = to_host(Z)
    lam = sum(4.0 / h ** 2 * np.sin(0.5 * np.pi / (k + 1)) ** 2 for k, h in zip(g.m, g.h))
    tol = 1e-12 + np.finfo(float).eps * sum(2.0 / h ** 2 for h in g.h) / lam
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))


@pytest.mark.parametrize("N", [33, 45, 66, 72, 99, 130, 250])
def test_vcycle_and_its_dot_products_with_a_short_last_slice(N):
    """Widths whose vector groups do not divide into slices: the V-cycle, and one
    and three PCG iterations from the dot products of its last sweep."""
    from paper_2511_06788_amd import ope
    p = W.wells_3d(m=13, N=N, seed=11)
    op = _op(p)
    R = np.random.default_rng(N).standard_normal((p.grid.n, N))
    ref = O.Hierarchy(op).vcycle(R)
    U = W.initial_block(p.grid.n, N, 5)
    say(f"mg short slice N={N}")
    with _ctx(p) as c:
        Z = empty_dev(p.grid.n, N)
        ope.ope_mg_vcycle(c.handle, to_dev(R), Z)
        assert np.max(np.abs(to_host(Z) - ref)) <= 1e-12 * np.max(np.abs(ref))
        for k in (1, 3):
            Yd = empty_dev(p.grid.n, N)
            ope.ope_source_solve(c.handle, to_dev(U), Yd, None, 1e-15, k, allow_maxit=True)
            Y_ref = O.pcg_source(op, U, None, tol=1e-15, max_iter=k)
            assert np.max(np.abs(to_host(Yd) - Y_ref)) <= 1e-12 * np.max(np.abs(Y_ref))


def test_vcycle_on_a_plane_of_more_than_4_gib():
    """A 2D block of 2^29 FP64 values and more takes 64-bit offsets: the same
    columns in a block half as wide, below the line, give the same V-cycle."""
    import torch
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid((2050, 2050))
    V = W.harmonic_potential(g, 100.0, (0.5, 0.5))
    gen = torch.Generator(device="cuda").manual_seed(3)
    R = torch.randn(g.n, 64, dtype=torch.float64, device="cuda", generator=gen)
    out = []
    for N in (64, 128):
        Rn = R if N == 64 else torch.cat([R, R.flip(1)], dim=1).contiguous()
        Z = torch.empty_like(Rn)
        say(f"mg vcycle 2050^2 N={N}")
        with ope.Context(g, V, N) as c:
            ope.ope_set_multigrid(c.handle, True)
            ope.ope_mg_vcycle(c.handle, Rn, Z)
        out.append(Z)
        del Rn
    scale = float(out[0].abs().max())
    assert float((out[1][:, :64] - out[0]).abs().max()) <= 1e-13 * scale
    assert float((out[1][:, 64:].flip(1) - out[0]).abs().max()) <= 1e-13 * scale


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("m,N", [((13, 13, 13), 2), ((26, 27, 25), 4)])
def test_step_ignores_what_an_earlier_vcycle_left_in_stopped_columns(m, N, precision):
    """A column below its target before the first iteration (an exact eigenvector
    beside rough ones) is skipped by the V-cycles' coarse levels; a V-cycle of a
    block of NaN before the step must not reach it.  The step equals a fresh
    context's bit for bit."""
    import torch
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid(m)
    mode = np.array([[1.0]])
    for k in g.m[::-1]:
        mode = np.kron(mode, np.sqrt(2.0 / (k + 1)) * np.sin(np.pi * np.arange(1, k + 1) / (k + 1))[:, None])
    rest = np.random.default_rng(N).standard_normal((g.n, N - 1))
    rest -= mode @ (mode.T @ rest)
    U0 = np.concatenate([mode, np.linalg.qr(rest)[0]], axis=1)
    dt = torch.float32 if precision else torch.float64
    out = []
    for poison in (False, True):
        say(f"stopped column after a NaN V-cycle m={m} N={N} precision={precision} poison={poison}")
        with ope.Context(g, np.zeros(g.n), N, precision=precision) as c:
            ope.ope_set_multigrid(c.handle, True)
            if poison:
                R = torch.full((g.n, N), float("nan"), dtype=dt, device="cuda")
                ope.ope_mg_vcycle(c.handle, R, torch.empty_like(R))
            U = torch.from_numpy(U0).to("cuda").to(dt).contiguous()
            info = ope.ope_step(c.handle, U, 1.0)
            out.append((U.cpu().numpy(), info.energy, info.residual, info.inner_iterations))
    assert np.all(np.isfinite(out[1][0])) and out[1][3] > 0
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


@pytest.mark.parametrize("m,N", [((97, 90), 128), ((200, 200), 65), ((500, 130), 40)])
def test_pcg_scalars_of_many_partial_rows(m, N):
    """Planes whose tiles give more partial sums than one work-group takes (the
    last two; the first is just below): one and three PCG iterations against the
    oracle's."""
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid(m)
    V = np.random.default_rng(N).uniform(0.0, 40.0, g.n)
    op = O.Operator(g.m, g.h, V)
    U = W.initial_block(g.n, N, 5)
    say(f"pcg scalars m={m} N={N}")
    with ope.Context(g, V, N) as c:
        ope.ope_set_multigrid(c.handle, True)
        for k in (1, 3):
            Yd = empty_dev(g.n, N)
            its = ope.ope_source_solve(c.handle, to_dev(U), Yd, None, 1e-15, k, allow_maxit=True)
            Y_ref = O.pcg_source(op, U, None, tol=1e-15, max_iter=k)
            assert its == k
            assert np.max(np.abs(to_host(Yd) - Y_ref)) <= 1e-12 * np.max(np.abs(Y_ref))


def test_pcg_scalars_of_a_large_plane_are_not_one_work_groups():
    """At 500^2, N = 128 the dot products' 4 MB of partial sums take about 15 us
    over the chip and 93 us through one compute unit; a third of that is the line."""
    import torch
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid((500, 500))
    N = 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    U = torch.linalg.qr(torch.randn(g.n, N, dtype=torch.float64, device="cuda", generator=gen))[0].contiguous()
    say("pcg scalars of a large plane")
    with ope.Context(g, np.zeros(g.n), N) as c:
        ope.ope_set_multigrid(c.handle, True)
        Y = torch.empty_like(U)
        ope.ope_source_solve(c.handle, U, Y, None, 1e-30, 2, allow_maxit=True)
        ope.ope_profile_begin(c.handle, ope.OPE_KERNEL_CG_REDUCE)
        ope.ope_source_solve(c.handle, U, Y, None, 1e-30, 12, allow_maxit=True)
        _, _, tags, ms = ope.ope_profile_end_launches(c.handle, 64)
    tags, ms = np.asarray(tags), np.asarray(ms)
    beta = [ms[tags == k][-1] for k in range(12)]
    assert min(beta) <= 0.031, beta


@pytest.mark.parametrize("m,N", [((5, 4, 700), 3), ((8, 8, 515), 8), ((3, 2, 1100), 16), ((16, 16, 300), 4)])
def test_vcycle_of_long_thin_grids(m, N):
    """Few tiles and many planes: more than 64 z ranges per tile, of one plane and
    more; the V-cycle and two PCG iterations from its dot products (the bounds of
    the fused coarse end's test)."""
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid(m)
    rng = np.random.default_rng(N)
    V = rng.uniform(0.0, 40.0, g.n)
    op = O.Operator(g.m, g.h, V)
    R = rng.standard_normal((g.n, N))
    ref = O.Hierarchy(op).vcycle(R)
    say(f"mg long thin grid m={m} N={N}")
    lam = sum(4.0 / h ** 2 * np.sin(0.5 * np.pi / (k + 1)) ** 2 for k, h in zip(g.m, g.h))
    tol = 1e-12 + np.finfo(float).eps * sum(2.0 / h ** 2 for h in g.h) / lam
    with ope.Context(g, V, N) as c:
        ope.ope_set_multigrid(c.handle, True)
        Z = empty_dev(g.n, N)
        ope.ope_mg_vcycle(c.handle, to_dev(R), Z)
        assert np.max(np.abs(to_host(Z) - ref)) <= tol * np.max(np.abs(ref))
        ope.ope_source_solve(c.handle, to_dev(R), Z, None, 1e-15, 2, allow_maxit=True)
        Y_ref = O.pcg_source(op, R, None, tol=1e-15, max_iter=2)
        assert np.max(np.abs(to_host(Z) - Y_ref)) <= tol * np.max(np.abs(Y_ref))


def test_vcycle_of_a_long_thin_grid_fills_the_chip():
    """One tile of 4000 planes: 64 z ranges leave three quarters of the compute units
    idle (0.225 ms a V-cycle, 0.158 with 512 work-groups of any size, 0.105 with the
    ranges that fill the chip once)."""
    import torch
    from paper_2511_06788_amd import ope
    g = W.unit_box_grid((8, 8, 4000))
    N = 8
    gen = torch.Generator(device="cuda").manual_seed(7)
    R = torch.randn(g.n, N, dtype=torch.float64, device="cuda", generator=gen)
    Z = torch.empty_like(R)
    say("mg long thin grid time")
    with ope.Context(g, np.zeros(g.n), N) as c:
        ope.ope_set_multigrid(c.handle, True)
        ope.ope_mg_vcycle(c.handle, R, Z)
        ope.ope_profile_begin(c.handle, ope.OPE_KERNEL_MG)
        for _ in range(10):
            ope.ope_mg_vcycle(c.handle, R, Z)
        _, _, _, ms = ope.ope_profile_end_launches(c.handle, 64)
    assert min(ms) <= 0.158, ms
