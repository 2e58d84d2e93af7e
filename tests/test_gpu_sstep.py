"""The s-step GCR cycles (directions built without inner products, one minimal-residual
solve per cycle) of the smoother and of the coarsest level, for every cycle length."""
import numpy as np
import pytest
import torch

from oracle import dwf_oracle as O
from paper_2004_07732_amd import inputs

pytestmark = pytest.mark.gpu

dwfmg = pytest.importorskip("paper_2004_07732_amd.dwfmg")


def T(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def pair(L, Ls, m, nvec, Lsc, seed, **kw):
    U = inputs.metropolis_u1(L, L, 6.0, 30, seed).U
    start = inputs.gaussian_field((nvec, L, L, 2), seed + 1)
    p = dwfmg.MGParams(nvec=[nvec], block=[(4, 4)], Ls_coarse=[Lsc], link_prec=[dwfmg.P_F64], vec_prec=[dwfmg.P_F64],
                       setup_iters=0, **kw)
    mg = dwfmg.MG(T(U), Ls, m, -1.0, p, [T(start)], max_nrhs=3)
    o = O.MG(U, Ls, m, -1.0, O.MGParams(levels=[O.LevelParams(nvec=nvec, block=(4, 4), Ls=Lsc, setup_iters=0)],
                                        smooth_iters=p.smooth_iters, coarsest_tol=p.coarsest_tol,
                                        coarsest_maxit=p.coarsest_maxit), [start])
    return mg, o


@pytest.mark.parametrize("steps,restart", [(1, 0), (2, 1), (5, 2), (7, 5), (13, 6), (7, 0), (15, 7), (16, 8)])
def test_smoother_cycle_lengths(steps, restart):
    """K-cycle in FP64 against the oracle for cycles of 1..8 steps, with a shorter last
    cycle where the length does not divide; three columns, the middle one zero.  Bar:
    the oracle's own coarsest CGNR to 1e-12 leaves 1e-10 at these condition numbers."""
    mg, o = pair(16, 4, 0.05, 4, 4, 900, smooth_iters=steps, smooth_restart=restart, coarsest_tol=1e-12,
                 coarsest_maxit=4000)
    o.params.smooth_restart = restart
    r = inputs.gaussian_field((3, 4, 16, 16, 2), 901)
    r[1] = 0.0
    got = mg.level_op(0, dwfmg.MG_OP_KCYCLE, T(r), 3).cpu().numpy()
    assert not got[1].any()
    for c in (0, 2):
        want = o.kcycle(0, r[c])
        assert np.linalg.norm(got[c] - want) < 1e-8 * np.linalg.norm(want)


def gcr(A, b, k, tol):
    """Restarted minimal residual over Krylov spaces of up to k steps, stopped at the first
    step at or below tol |b| (dense least squares on an orthonormal basis)."""
    x, r, nb = np.zeros_like(b), b.copy(), np.linalg.norm(b)
    while True:
        q = [r / np.linalg.norm(r)]
        for j in range(1, k + 1):
            Q = np.stack(q, 1)
            y = np.linalg.lstsq(A @ Q, r, rcond=None)[0]
            res = r - A @ (Q @ y)
            if np.linalg.norm(res) <= tol * nb:
                return x + Q @ y
            w = A @ q[-1]
            for _ in range(2):
                w = w - Q @ (Q.conj().T @ w)
            q.append(w / np.linalg.norm(w))
        x, r = x + Q @ y, res


@pytest.mark.parametrize("restart", [1, 2, 3, 4, 5, 6, 7, 8])
def test_coarsest_cycles_stop_at_the_step(restart):
    """Coarsest GCR to a loose tolerance, which most columns meet inside a cycle: the
    correction is that of the step that met it, per column."""
    tol = 0.2
    mg, o = pair(16, 4, 0.05, 4, 2, 910, smooth_iters=0, coarsest_solver=dwfmg.COARSEST_GCR,
                 coarsest_restart=restart, coarsest_tol=tol)
    A = O.assemble(lambda v: o.A(1, v), (2, 4, 4, 8))
    r = inputs.gaussian_field((3, 4, 16, 16, 2), 911)
    r[2] *= 1e-6
    got = mg.level_op(0, dwfmg.MG_OP_KCYCLE, T(r), 3).cpu().numpy()
    for c in range(3):
        rc = o.restrict(0, r[c])
        want = o.prolong(0, gcr(A, rc.reshape(-1), restart, tol).reshape(rc.shape))
        assert np.linalg.norm(got[c] - want) < 1e-9 * np.linalg.norm(want)


def test_exhausted_krylov_space():
    """A coarse space smaller than the cycle (one coarse site, 2 slices, 4 components: the
    directions become dependent): dependent directions are dropped, the solve is exact."""
    mg, o = pair(4, 4, 0.1, 2, 2, 920, smooth_iters=0, coarsest_solver=dwfmg.COARSEST_GCR, coarsest_restart=8,
                 coarsest_tol=1e-12)
    A = O.assemble(lambda v: o.A(1, v), (2, 1, 1, 4))
    r = inputs.gaussian_field((1, 4, 4, 4, 2), 921)
    got = mg.level_op(0, dwfmg.MG_OP_KCYCLE, T(r), 1).cpu().numpy()[0]
    rc = o.restrict(0, r[0])
    want = o.prolong(0, np.linalg.solve(A, rc.reshape(-1)).reshape(rc.shape))
    assert np.linalg.norm(got - want) < 1e-9 * np.linalg.norm(want)
