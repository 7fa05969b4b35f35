"""The sizes where a launch rule changes its shape: each kernel against the oracle or a plain
64-bit result at the edges and remainders of its tiles."""
import math

import numpy as np
import pytest
import torch

from henry_inputs import draw_theta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    import paper_2403_17018_amd as P
    h = P.Henry(0)
    yield h
    h.close()


def _cu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("m", [(1, 2), (3, 15), (16, 17), (33, 64), (65, 255), (256, 1023), (1024, 1025), (4096, 4099)])
def test_moments_at_every_row_width(hx, m):
    """Rows of m samples are shared by 1 .. 64 threads or a block, with remainders: level and
    cell moments against numpy.  Bound: a sum of m terms in any order is off by at most
    (m - 1) eps of the sum of magnitudes; mean and squared deviations take a few such sums."""
    import paper_2403_17018_amd as P
    rng = np.random.default_rng(5)
    grids = [P.grid(6, 3, 1), P.grid(12, 6, 1)]
    gf = [rng.normal(3.0, 1.0, k) for k in m]
    gc = [None, rng.normal(2.5, 1.0, m[1])]
    cf = [rng.uniform(size=(g.ny, g.nx, k)) for g, k in zip(grids, m)]
    cc = [None, rng.uniform(size=(3, 6, m[1]))]
    cu = lambda a: None if a is None else _cu(a)
    out = hx.mlmc_estimate(grids, [cu(a) for a in gf], [cu(a) for a in gc], [cu(a) for a in cf], [cu(a) for a in cc])
    Y = [gf[0], gf[1] - gc[1]]
    var = lambda a: a.var(axis=-1, ddof=1) if a.shape[-1] > 1 else np.zeros(a.shape[:-1])
    eps = 2.3e-16 * (max(m) + 10)
    assert abs(out["mean"] - sum(y.mean() for y in Y)) <= 8 * eps * sum(np.abs(y).mean() for y in Y)
    for v, y in zip(out["V"], Y):
        assert abs(v - var(y)) <= 8 * eps * (np.abs(y) ** 2).mean() * len(y) / max(1, len(y) - 1)
    up = lambda a: a.repeat(2, 0).repeat(2, 1)
    mean = up(cf[0].mean(-1)) + cf[1].mean(-1) - up(cc[1].mean(-1))
    vf = up(var(cf[0])) + var(cf[1]) - up(var(cc[1]))
    assert np.abs(out["mean_field"].cpu().numpy() - mean).max() <= 8 * eps * 3
    assert np.abs(out["var_field"].cpu().numpy() - vf).max() <= 8 * eps * 3 * 2


@pytest.mark.parametrize("nx,ny,S", [
    *[(nx, ny, S) for nx, ny in ((6, 3), (34, 17), (64, 32)) for S in (1, 3, 16, 37, 64, 130)],
    (1030, 515, 1), (1030, 515, 3), (260, 130, 16),    # 1024, 340 and 64 cells a block
    (400, 200, 1), (300, 150, 3),                      # 128 and 85
])
@pytest.mark.parametrize("model", ["kl", "paper"])
def test_fields_at_block_edges(hx, nx, ny, S, model):
    """4 * (256 / min(S, 64)) cells a block, of few samples halved towards 32 while fewer than 512
    blocks are left, with remainders: phi, K and u_in against the oracle.  Bound: 8 + 8 products and
    sums, and exp's argument (about 21) carried to K."""
    import paper_2403_17018_amd as P
    from oracle import henry as H
    th = draw_theta(31, S, level=1)
    prob, pro = (P.paper_problem(), H.paper_problem()) if model == "paper" else (P.problem(), H.Problem())
    phi, K, u = (t.cpu().numpy() for t in hx.sample_fields(_cu(th), P.grid(nx, ny, 4), prob))
    for s in range(S):
        a, b, c = H.sample_fields(pro, H.Grid(nx, ny, 4), th[s])
        assert np.abs(phi[..., s].ravel() - np.ravel(a)).max() <= 1e-13
        assert (np.abs(K[..., s].ravel() - np.ravel(b)) <= 1e-12 * np.abs(np.ravel(b))).all()
        assert abs(u[s] - c) <= 1e-15 * abs(c)


@pytest.mark.parametrize("n_phi,n_logK", [(0, 0), (2, 0), (0, 3), (4, 5)])
def test_fields_with_fewer_modes(hx, n_phi, n_logK):
    """Modes beyond the problem's counts contribute nothing: equal to the full set with their
    coefficients at zero, up to the sign of a zero."""
    import paper_2403_17018_amd as P
    th = draw_theta(32, 5)
    z = th.copy()
    z[:, n_phi:4] = 0.0
    z[:, 4 + n_logK:12] = 0.0
    g = P.grid(20, 10, 1)
    a = hx.sample_fields(_cu(th), g, P.problem(n_kl_phi=n_phi, n_kl_logK=n_logK))
    b = hx.sample_fields(_cu(z), g, P.problem())
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("S", [1, 17, 130])
@pytest.mark.parametrize("nx,ny,coarse,sweeps", [
    (16, 8, 8, (1, 2)),      # the coarsest grid alone
    (32, 16, 8, (1, 1)),     # one smoothed grid with it
    (64, 32, 8, (2, 2)),     # two, the finest of 512 cells, two pre-smoothing sweeps
    (64, 32, 4, (1, 2)),     # three
    (128, 64, 2, (1, 2)),    # three in one launch, more above
    (40, 20, 10, (1, 2)),    # a coarsest grid of 50 cells, odd rows
])
def test_coarse_grids_in_one_launch(hx, prec, S, nx, ny, coarse, sweeps):
    """The multigrid's coarse end (state restriction, Jacobians, inverse of the coarsest operator
    and the cycle) in launches of one workgroup per sample: the solve against the oracle (1e-8,
    the workload's bound), and the preconditioner's strength, which a wrong coarse correction
    would take away: at most 1.35 BiCGStab iterations per Newton iteration on average (1.00 to
    1.13 with a launch per grid and pass)."""
    import paper_2403_17018_amd as P
    from tests.oracle_runs import oracle_batch, rel_inf
    th = draw_theta(41, S, level=1)
    g = P.grid(nx, ny, 3)
    kw = dict(T=36000.0 * 3 / (3 * ny))
    o = P.solver_opts(mg_precision=prec, coarse_nx=coarse, coarse_ny=max(1, coarse // 2), nu_pre=sweeps[0],
                      nu_post=sweeps[1], step_graphs=0)
    r = hx.solve(_cu(th), g, P.problem(**kw), o)
    assert r.nfailed == 0
    pick = sorted({0, S // 2, S - 1})
    ref = oracle_batch(th[pick], nx, ny, 3, kw)
    assert rel_inf(r.c_T.permute(2, 0, 1).cpu().numpy()[pick], ref["c"]).max() <= 1e-8
    newton, bicg = r.stats[:, 0].sum().item(), r.stats[:, 1].sum().item()
    assert bicg <= 1.35 * newton, (newton, bicg)


def test_coarse_grids_in_one_launch_transposed(hx):
    """The transposed cycle of the adjoint through three smoothed grids in one launch: the
    gradient against the one with the pivoted coarse solver and a launch per pass."""
    import paper_2403_17018_amd as P
    th = _cu(draw_theta(42, 5, level=1))
    g, prob = P.grid(64, 32, 6), P.problem(T=2250.0)
    tight = dict(newton_tol=1e-13, krylov_rtol=1e-12, krylov_maxit=200, newton_maxit=60, krylov_rtol_adjoint=1e-12)
    ref = hx.adjoint(th, g, prob, P.solver_opts(coarse_solver=2, **tight), checkpoint_every=4)[1]
    for cnx in (4, 8):
        for prec in (64, 32):
            gr = hx.adjoint(th, g, prob, P.solver_opts(coarse_nx=cnx, coarse_ny=cnx // 2, mg_precision=prec, **tight),
                            checkpoint_every=4)[1]
            assert (gr - ref).abs().max() <= 1e-9 * ref.abs().max(), (cnx, prec)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("nx,ny,S,opts", [
    (16, 8, 1, {}),                                    # the coarsest grid alone
    (16, 8, 17, dict(coarse_nx=12, coarse_ny=6)),      # no coarse grid: sweeps on the fine one
    (32, 16, 33, dict(nu_pre=2)),                      # one smoothed grid in the launch
    (64, 32, 5, dict(nu_post=1)),                      # two, 561 and 153 vertices
    (64, 32, 5, dict(coarse_nx=4, coarse_ny=2)),       # two of the three coarse grids
    (40, 24, 5, dict(coarse_nx=10, coarse_ny=6)),      # 77 vertices are too many to invert: sweeps
    (36, 20, 5, dict(coarse_nx=9, coarse_ny=5)),       # a coarsest grid of 60 vertices, odd sides
])
def test_vertex_coarse_grids_in_one_launch(hx, prec, nx, ny, S, opts):
    """The vertex-centred cycle's coarse end in launches of one workgroup per sample, against the
    vertex oracle (1e-8, the workload's bound), and its strength where there is a cycle: at most
    1.35 BiCGStab iterations per Newton iteration (1.00 to 1.05 with a launch per pass)."""
    import paper_2403_17018_amd as P
    from oracle import henry as H
    from oracle import vertex as V
    import dataclasses
    th = draw_theta(43, S, level=1)
    steps, T = 3, 3 * 64.0 * 8 / ny
    r = hx.vc_solve(_cu(th), P.grid(nx, ny, steps), P.paper_problem(T=T),
                    P.solver_opts(mg_precision=prec, krylov_maxit=300, **opts), want_p=True)
    assert r.nfailed == 0
    for s in sorted({0, S - 1}):
        ref = V.solve_sample(dataclasses.replace(H.paper_problem(), T=T), H.Grid(nx, ny, steps), th[s])
        c = r.c_T[..., s].cpu().numpy().ravel()
        assert np.abs(c - np.ravel(ref.c)).max() <= 1e-8 * np.abs(ref.c).max()
    if opts.get("coarse_nx", 8) not in (10, 12):
        newton, bicg = r.stats[:, 0].sum().item(), r.stats[:, 1].sum().item()
        assert bicg <= 1.35 * newton, (newton, bicg)


@pytest.mark.parametrize("nx,ny,S,solver", [
    (2, 2, 1, 2),        # one panel, wider than the matrix
    (3, 3, 3, 2),        # 18 unknowns: a last panel of 2
    (4, 4, 2, 1), (16, 8, 17, 1), (32, 16, 130, 1),
    (9, 19, 2, 2),       # the longer side second
    (40, 19, 2, 2),      # the widest band
    (60, 9, 3, 2),
    (32, 32, 2, 1),      # two rows a lane (FP32 operators only)
])
def test_pivoted_solvers_at_panel_edges(hx, nx, ny, S, solver):
    """LU with partial pivoting, plain and transposed, on random blocks whose first cell has a zero
    pivot: normwise backward error at most 200 eps (n eps growth of a stable elimination, with
    its constants) and the error against numpy within its condition."""
    import paper_2403_17018_amd as P
    from tests.test_gpu_kernels import _blocks_to_sparse
    rng = np.random.default_rng(nx * 100 + ny)
    J = rng.normal(size=(20, ny, nx, S))
    J[4:8, :, 0] = J[8:12, :, -1] = 0.0
    J[12:16, 0] = J[16:20, -1] = 0.0
    J[0:4, 0, 0] = np.array([0.0, 1.0, 1.0, 0.0])[:, None]
    b = rng.normal(size=(2, ny, nx, S))
    for prec in ((32,) if (nx, ny) == (32, 32) else (64, 32)):
        if prec == 32:
            J, b = J.astype(np.float32).astype(float), b.astype(np.float32).astype(float)
        for tr in (False, True):
            x = hx.coarse_solve(_cu(J), _cu(b), P.grid(nx, ny, 1), solver, prec, tr).cpu().numpy()
            for s in sorted({0, S - 1}):
                A = _blocks_to_sparse(J[..., s], nx, ny).toarray()
                A = A.T if tr else A
                vec = lambda a: np.stack([a[0, ..., s].ravel(), a[1, ..., s].ravel()], axis=1).ravel()
                bs, xs = vec(b), vec(x)
                eps = 2.2e-16 if prec == 64 else 6e-8   # FP32: rounding of the result alone
                berr = np.abs(A @ xs - bs).max() / (np.abs(A).sum(1).max() * np.abs(xs).max() + np.abs(bs).max())
                assert berr <= 200 * eps, (prec, tr, s, berr)
                ref = np.linalg.solve(A, bs)
                assert np.abs(xs - ref).max() <= 1000 * eps * np.linalg.cond(A, np.inf) * np.abs(ref).max()


@pytest.mark.parametrize("what", ["row", "column"])
@pytest.mark.parametrize("nx,ny,solver", [(8, 4, 1), (8, 4, 2), (3, 3, 2), (32, 16, 1)])
def test_pivoted_solvers_of_a_singular_operator(hx, nx, ny, solver, what):
    """One sample's operator has an unknown without an equation, or without an entry in any: its
    solution is not finite, the others' are."""
    import paper_2403_17018_amd as P
    rng = np.random.default_rng(9)
    J = rng.normal(size=(20, ny, nx, 3))
    J[4:8, :, 0] = J[8:12, :, -1] = 0.0
    J[12:16, 0] = J[16:20, -1] = 0.0
    i, j = nx // 2, ny // 2
    for k, (di, dj) in enumerate(((0, 0), (1, 0), (-1, 0), (0, 1), (0, -1))):
        if what == "row":
            J[4 * k:4 * k + 2, j, i, 1] = 0.0
        elif 0 <= i + di < nx and 0 <= j + dj < ny:   # the rows of which (i, j) is neighbour k
            J[[4 * k, 4 * k + 2], j + dj, i + di, 1] = 0.0
    b = _cu(rng.normal(size=(2, ny, nx, 3)))
    for prec in (64, 32):
        for tr in (False, True):
            x = hx.coarse_solve(_cu(J), b, P.grid(nx, ny, 1), solver, prec, tr)
            assert torch.isfinite(x[..., [0, 2]]).all(), (prec, tr)
            assert not torch.isfinite(x[..., 1]).all(), (prec, tr)


@pytest.mark.parametrize("nx,ny,S,opts", [
    (64, 32, 64, dict()),
    (64, 32, 129, dict(nu_pre=2, nu_post=1)),
    (64, 32, 130, dict(nu_pre=1, nu_post=0)),
    (64, 32, 129, dict(fuse_prolong=0)),
    (128, 64, 33, dict(mg_cycle=2)),
    (128, 64, 33, dict(coarse_nx=16, coarse_ny=8, coarse_solver=2)),
    (68, 34, 115, dict()),                                      # 34x17 cells: no single launch, band LU
    (34, 17, 454, dict()),                                      # the fine grid is the coarsest
    (64, 32, 289, dict()),                                      # marched through: one strip, odd batch
    (32, 16, 1153, dict()),
    (144, 72, 57, dict()),                                      # several strips
    (128, 64, 73, dict(mg_cycle=2)),
    (512, 256, 5, dict()),                                      # many strips and segments, part of a block
    (64, 32, 641, dict(mg_precision=32)),
    (144, 72, 127, dict(mg_precision=32)),
    (512, 256, 11, dict(mg_precision=32)),
    (64, 32, 129, dict(problem=dict(recharge_omega=2e-3, q_in_amp=0.3, right_c_dirichlet=1))),
])
def test_rows_formed_from_the_state(hx, nx, ny, S, opts):
    """A batch of at least 2^17 cell-samples forms its operators' rows from the state, and one of at
    least 9 * 2^16 (FP32: 5 * 2^18) marches through the grid with several passes a launch; the same
    samples alone read stored Jacobians.  Both solve the same equations to the Newton tolerance
    (1e-8 on the state, the workload's bound), with as strong a preconditioner: at most 5 % and
    one BiCGStab iteration a sample more."""
    import paper_2403_17018_amd as P
    opts = dict(opts)
    kw = dict(opts.pop("problem", {}), T=36000.0 * 4 / (3 * ny))
    th = draw_theta(43, S, level=1)
    g = P.grid(nx, ny, 4)
    o = P.solver_opts(**{"step_graphs": 0, **opts})   # (not the one launch a step of small grids)
    pick = [0, S // 2, S - 1]
    a = hx.solve(_cu(th), g, P.problem(**kw), o, want_c=True, want_p=True)
    b = hx.solve(_cu(th[pick]), g, P.problem(**kw), o, want_c=True, want_p=True)
    assert a.nfailed == 0 and b.nfailed == 0
    for u, v in ((a.c_T, b.c_T), (a.p_T, b.p_T)):
        u, v = u.permute(2, 0, 1)[pick], v.permute(2, 0, 1)
        assert ((u - v).abs().amax() / v.abs().amax()).item() <= 1e-8
    ia, ib = a.stats[pick, 1].cpu().numpy(), b.stats[:, 1].cpu().numpy()
    assert (ia <= 1.05 * ib + 1).all(), (ia, ib)


def test_fp32_solve_and_adjoint_on_one_plan(hx):
    """A solve (whose products read the FP32 Jacobian) and an adjoint (whose products read the FP64
    one) of the same shape share a plan: each must come out as on a context of its own, in either
    order, to the linear solves' tolerance (1e-8 on the state, the workload's bound)."""
    import paper_2403_17018_amd as P
    th = _cu(draw_theta(47, 20, level=0))
    g, pr = P.grid(80, 40, 12), P.problem(T=3600.0)              # above one-launch steps' cells
    o = P.solver_opts(mg_precision=32)

    def close(u, v):
        return ((u - v).abs().amax() / v.abs().amax()).item() <= 1e-8

    h = P.Henry(0)
    s0 = h.solve(th, g, pr, o, want_c=True).c_T.clone()
    h.close()
    h = P.Henry(0)
    q0, g0 = [t.clone() for t in h.adjoint(th, g, pr, o)[:2]]
    s1 = h.solve(th, g, pr, o, want_c=True).c_T.clone()
    q1, g1 = [t.clone() for t in h.adjoint(th, g, pr, o)[:2]]
    h.close()
    assert close(s1, s0) and close(q1, q0) and close(g1, g0)


@pytest.mark.parametrize("nx,ny,S,opts", [
    (4, 2, 3, dict(coarse_nx=2, coarse_ny=1)),
    (16, 8, 1, dict()),
    (32, 16, 9, dict()),
    (32, 16, 130, dict(nu_pre=2, nu_post=1)),
    (32, 16, 17, dict(coarse_nx=4, coarse_ny=2)),               # three smoothed grids
    (40, 20, 20, dict()),                                       # a coarsest grid of 50 cells, idle threads
    (24, 12, 33, dict()),                                       # a coarsest grid of 18 cells, half the threads idle
    (20, 10, 33, dict()),                                       # the coarsest grid alone below the fine one, 50 cells
    (48, 24, 7, dict(nu_pre=3, nu_post=1)),                     # two cells of a colour a thread
    (64, 32, 40, dict()),
    (64, 32, 300, dict()),                                      # more samples than workgroups at once
    (64, 32, 5, dict(coarse_nx=4, coarse_ny=2)),                # four smoothed grids
    (32, 16, 12, dict(newton_predict=0.0, newton_jac_reuse=0.0)),
    (32, 16, 12, dict(newton_dc_max=0.05)),                     # damped updates
    (32, 16, 12, dict(newton_maxit=1)),                         # not converged: status 1
    (32, 16, 12, dict(krylov_maxit=1)),
    (64, 32, 12, dict(problem=dict(recharge_omega=2e-3, q_in_amp=0.3, right_c_dirichlet=1))),
    (32, 16, 12, dict(problem=dict(field_model=1))),
    (32, 16, 9, dict(mg_precision=32)),
    (48, 24, 65, dict(mg_precision=32)),
])
def test_small_grids_in_one_launch_a_step(hx, nx, ny, S, opts):
    """Grids of up to 2048 cells solve a step in one launch, a workgroup per sample; step_graphs
    0 takes them launch by launch.  Both solve the same equations: the state of the solved samples to 1e-8 (the
    workload's bound), the same status, and at most 15 % (and 3) more BiCGStab iterations a sample, as a chord
    step's fine rows and coarse correction are not of the same state."""
    import paper_2403_17018_amd as P
    opts = dict(opts)
    kw = dict(opts.pop("problem", {}), T=36000.0 * 6 / (3 * max(ny, 8)))
    th = _cu(draw_theta(51, S, level=0))
    g = P.grid(nx, ny, 6)
    reads = [hx.profile_read()["host_sync"][0]]
    a = hx.solve(th, g, P.problem(**kw), P.solver_opts(**opts), want_c=True, want_p=True)
    reads.append(hx.profile_read()["host_sync"][0])
    b = hx.solve(th, g, P.problem(**kw), P.solver_opts(step_graphs=0, **opts), want_c=True, want_p=True)
    reads.append(hx.profile_read()["host_sync"][0])
    assert reads[1] - reads[0] <= 1 and reads[2] - reads[1] > 6, reads   # no read within steps but launch by launch
    assert torch.equal(a.status, b.status)
    ok = b.status == 0
    assert ok.any() or opts.get("newton_maxit") == 1
    for u, v in ((a.c_T, b.c_T), (a.p_T, b.p_T)):
        u, v = u[..., ok], v[..., ok]
        assert u.numel() == 0 or ((u - v).abs().amax() / v.abs().amax()).item() <= 1e-8
    ia, ib = a.stats[:, 1].sum().item(), b.stats[:, 1].sum().item()
    assert ia <= 1.15 * ib + 3 * S, (ia, ib)


def test_memory_for_compaction_only_where_it_can_happen():
    """A shape whose steps never move samples to a smaller batch (fewer than 3 * 2^19 cell-samples, or
    one launch a step) holds one plan, not two; a later call that may (launch by launch) gets its
    second then.  700 samples of 64x32 cells are below that number, 800 above."""
    import paper_2403_17018_amd as P
    g, pr = P.grid(64, 32, 1), P.problem(T=375.0)
    used = {}
    for S, graphs in ((700, (0,)), (800, (0,)), (800, (1,)), (800, (1, 0))):
        th = _cu(draw_theta(74, S, level=0))
        h = P.Henry(0)
        for sg in (0, 1):   # the kernels' own memory (scratch of their queue)
            h.solve(th[:2].contiguous(), g, pr, P.solver_opts(step_graphs=sg), want_c=False)
        torch.cuda.synchronize()
        m0 = torch.cuda.mem_get_info()[0]
        for sg in graphs:
            assert h.solve(th, g, pr, P.solver_opts(step_graphs=sg), want_c=False).nfailed == 0
        torch.cuda.synchronize()
        used[S, graphs] = m0 - torch.cuda.mem_get_info()[0]
        h.close()
    assert used[700, (0,)] < 0.6 * used[800, (0,)], used
    assert used[800, (1,)] < 0.6 * used[800, (0,)], used
    assert used[800, (1, 0)] > 0.9 * used[800, (0,)], used


@pytest.mark.parametrize("tol", [1e-9, 1e-6, 1e-4])
def test_one_launch_steps_keep_operators_up_to_the_option(hx, tol):
    """newton_jac_reuse means its value in one-launch steps too: at the Newton tolerance no iteration
    follows an update of that size, so every operator is fresh, as with 0."""
    import paper_2403_17018_amd as P
    th = _cu(draw_theta(73, 40, level=0))
    g, pr = P.grid(32, 16, 6), P.problem(T=4500.0)
    a, b = [hx.solve(th, g, pr, P.solver_opts(newton_tol=tol, newton_predict=0.0, newton_jac_reuse=r), want_p=True)
            for r in (tol, 0.0)]
    assert torch.equal(a.stats, b.stats) and torch.equal(a.c_T, b.c_T) and torch.equal(a.p_T, b.p_T)
