"""GPU discrete adjoint: dQ/dtheta against the oracle's adjoint and against central
finite differences (absolute step h = 1e-6 per component) computed with the GPU
forward solve, all perturbed copies in one batch.

Bar (the workload's): max_k |g_adj - g_FD| <= 1e-6 * max_k |g_FD| per sample."""
import os

import numpy as np
import pytest
import torch

from henry_inputs import WORKLOADS, draw_theta, level_grid

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")
TIGHT = dict(newton_tol=1e-13, krylov_rtol=1e-12, krylov_maxit=200, newton_maxit=60)


@pytest.fixture(scope="module")
def hx():
    import paper_2403_17018_amd as P
    h = P.Henry(0)
    yield h
    h.close()


def _cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _oracle_adjoint(th, nx, ny, nsteps, T):
    """Oracle adjoint in a child interpreter (the test process has the GPU open)."""
    import json
    import subprocess
    import sys
    import tempfile
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = f"""
import sys, json, numpy as np
sys.path.insert(0, {root!r})
from oracle import henry as H, adjoint as A
th = np.array(json.loads(sys.argv[1]))
pr = H.Problem(T={T}); g = H.Grid({nx}, {ny}, {nsteps})
out = [A.adjoint_gradient(pr, g, t) for t in th]
print(json.dumps([[q, list(gr)] for q, gr in out]))
"""
    r = subprocess.run([sys.executable, "-c", code, json.dumps(th.tolist())], capture_output=True, text=True,
                       check=True)
    out = json.loads(r.stdout)
    return np.array([o[0] for o in out]), np.array([o[1] for o in out])


def _fd(hx, th, g, prob, opts, h=1e-6):
    """Central differences of Q for every sample and component, one batched GPU solve."""
    S = th.shape[0]
    pert = np.repeat(th[:, None, None, :], 2, axis=1).repeat(13, axis=2)   # [S, 2, 13, 13]
    for k in range(13):
        pert[:, 0, k, k] += h
        pert[:, 1, k, k] -= h
    r = hx.solve(_cu(pert.reshape(-1, 13)), g, prob, opts, want_c=False)
    assert r.nfailed == 0
    q = r.qoi.cpu().numpy().reshape(S, 2, 13)
    return (q[:, 0] - q[:, 1]) / (2 * h)


@pytest.mark.parametrize("shape", [(32, 16, 12, 9000.0, 5, 64), (48, 24, 10, 7500.0, 4, 64),
                                   (48, 24, 10, 7500.0, 4, 32)])
def test_adjoint_matches_oracle_and_fd(hx, shape):
    """Two shapes with FP64 multigrid, one with the FP32 multigrid preconditioner in both
    the forward and the transposed solves."""
    import paper_2403_17018_amd as P
    nx, ny, nsteps, T, ck, prec = shape
    th = draw_theta(21, 6, level=1)
    prob = P.problem(T=T)
    opts = P.solver_opts(mg_precision=prec, **TIGHT)
    g = P.grid(nx, ny, nsteps)
    q, gr, st, nf = hx.adjoint(_cu(th), g, prob, opts, checkpoint_every=ck)
    assert nf == 0
    q, gr = q.cpu().numpy(), gr.cpu().numpy()
    qo, go = _oracle_adjoint(th, nx, ny, nsteps, T)
    assert np.abs(q - qo).max() <= 1e-10 * np.abs(qo).max()
    for s in range(th.shape[0]):
        assert np.abs(gr[s] - go[s]).max() <= 1e-7 * np.abs(go[s]).max(), s
    fd = _fd(hx, th, g, prob, opts)
    for s in range(th.shape[0]):
        assert np.abs(gr[s] - fd[s]).max() <= 1e-6 * np.abs(fd[s]).max(), (s, gr[s], fd[s])


def test_adjoint_checkpoint_interval_does_not_change_gradient(hx):
    import paper_2403_17018_amd as P
    th = draw_theta(22, 4)
    g = P.grid(32, 16, 9)
    prob = P.problem(T=36000.0 * 9 / 48)
    opts = P.solver_opts(**TIGHT)
    ref = hx.adjoint(_cu(th), g, prob, opts, checkpoint_every=9)[1].cpu().numpy()
    for ck in (1, 2, 4):
        gr = hx.adjoint(_cu(th), g, prob, opts, checkpoint_every=ck)[1].cpu().numpy()
        assert np.array_equal(gr, ref), ck


def test_adjoint_level3_full_batch():
    """256x128 cells, 384 steps, 256 samples of seed 4, checkpoints every 32 steps (default
    solver tolerances, as benchmarked): samples 0, 108 and 255 against the stored oracle
    adjoint, samples 0..3 against central differences from batched GPU forward solves."""
    import paper_2403_17018_amd as P
    w = WORKLOADS["c5_adjoint_level3"]
    th = draw_theta(w["seed"], w["nsamples"], level=w["level"])
    g = P.grid(*level_grid(w["level"]))
    h = P.Henry(0)
    q, gr, st, nf = h.adjoint(_cu(th), g, checkpoint_every=w["checkpoint_every"])
    assert nf == 0
    gr = gr.cpu().numpy()
    for s in (0, 108, 255):      # the first, the smallest recharge zeta and the last sample
        z = np.load(os.path.join(GOLD, f"oracle_c5_adjoint_s{s}.npz"))
        assert np.array_equal(z["theta"], th[s])
        assert abs(q[s].item() - float(z["qoi"])) <= 1e-8 * abs(float(z["qoi"])), s
        assert np.abs(gr[s] - z["grad"]).max() <= 1e-6 * np.abs(z["grad"]).max(), s
    fd = _fd(h, th[:4], g, P.problem(), P.solver_opts(**TIGHT))
    for s in range(4):
        assert np.abs(gr[s] - fd[s]).max() <= 1e-6 * np.abs(fd[s]).max(), (s, gr[s], fd[s])
    h.close()


@pytest.mark.parametrize("nx,ny,S,T", [(64, 32, 8, 6000.0),      # forward steps a launch each
                                       (80, 40, 8, 2400.0),      # of captured iterations
                                       (80, 40, 48, 2400.0)])    # whose rows are formed from the state
def test_adjoint_with_graphs_equals_eager(hx, nx, ny, S, T):
    """Forward and transposed BiCGStab iterations replayed from hipGraphs (alternating in the
    reverse sweep) give bitwise the eager gradient."""
    import paper_2403_17018_amd as P
    th = draw_theta(23, S)
    g = P.grid(nx, ny, 8)
    prob = P.problem(T=T)
    a = hx.adjoint(_cu(th), g, prob, P.solver_opts(use_graphs=0), checkpoint_every=3)
    b = hx.adjoint(_cu(th), g, prob, P.solver_opts(use_graphs=1), checkpoint_every=3)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_adjoint_first_guess_changes_only_the_path(hx):
    """Transposed solves started from 0, from the later step's adjoint or from its linear
    extrapolation reach the same gradient when the solves are tight."""
    import paper_2403_17018_amd as P
    th = draw_theta(23, 5, level=1)
    g = P.grid(48, 24, 10)
    prob = P.problem(T=7500.0)
    out = []
    for guess in (0, 1, 2):
        opts = P.solver_opts(adjoint_guess=guess, krylov_rtol_adjoint=1e-12, **TIGHT)
        q, gr, st, nf = hx.adjoint(_cu(th), g, prob, opts, checkpoint_every=3)
        assert nf == 0
        out.append(gr.cpu().numpy())
    for gr in out[1:]:
        for s in range(th.shape[0]):
            assert np.abs(gr[s] - out[0][s]).max() <= 1e-9 * np.abs(out[0][s]).max(), s
    with pytest.raises(P.HenryError):
        hx.adjoint(_cu(th), g, prob, P.solver_opts(adjoint_guess=3))


def test_autograd_function_matches_adjoint_oracle_and_fd(hx):
    """torch.autograd through SaltMassQoI: the vector-Jacobian product with a weight vector w
    equals w[:, None] * dQ/dtheta of the adjoint call, the oracle adjoint (1e-7) and batched
    central differences (1e-6); without requires_grad only the forward solve runs (same Q)."""
    import paper_2403_17018_amd as P
    nx, ny, nsteps, T = 32, 16, 10, 7500.0
    th = draw_theta(24, 4, level=1)
    prob = P.problem(T=T)
    opts = P.solver_opts(**TIGHT)
    g = P.grid(nx, ny, nsteps)
    theta = _cu(th).requires_grad_(True)
    q = P.salt_mass_qoi(hx, theta, g, prob, opts, checkpoint_every=4)
    assert q.requires_grad and q.shape == (4,)
    w = torch.tensor([1.0, -2.0, 0.5, 3.0], dtype=torch.float64, device=q.device)
    (gt,) = torch.autograd.grad((w * q).sum(), theta)
    q2, gr, st, nf = hx.adjoint(_cu(th), g, prob, opts, checkpoint_every=4)
    assert nf == 0 and torch.equal(q.detach(), q2)
    assert torch.equal(gt, w[:, None] * gr)
    gr = gr.cpu().numpy()
    qo, go = _oracle_adjoint(th, nx, ny, nsteps, T)
    fd = _fd(hx, th, g, prob, opts)
    for s in range(4):
        assert np.abs(gr[s] - go[s]).max() <= 1e-7 * np.abs(go[s]).max(), s
        assert np.abs(gr[s] - fd[s]).max() <= 1e-6 * np.abs(fd[s]).max(), s
    q3 = P.salt_mass_qoi(hx, _cu(th), g, prob, opts)
    assert not q3.requires_grad
    assert torch.allclose(q3, q2, rtol=1e-12, atol=0)
