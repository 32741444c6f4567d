"""What one BiCGstab step leaves behind: |r^|^2 as accurate as the inner format
allows, and no reliable update that delta does not ask for.

At kappa << 1 the operator is close to 1, so one step removes almost all of
the residual: |r0| : |s| : |r| are about 1 : 8e-4 : 1e-6 at kappa 0.007.

Bound on |r|^2 (u: half a unit of the inner format): s = r0 - alpha v and
r = s - omega t round by up to 2u |r0| and 2u |s|, and so do v and t, which
enters |r|^2 twice: 8u (|r0| / |s| + |s| / |r|), and as much again for the FP64
oracle where the inner format is FP64 itself."""
import numpy as np
import pytest

import oracle
import paper_0911_3191_amd as wd
import wdinputs
from gpu_helpers import DEV, Setup

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DIMS, NRHS = (4, 4, 4, 4), 8


def one_step(U, kappa, b):
    """|r0|, |s|, |r| of the first BiCGstab step on b / |b|, r~ = r0, in FP64."""
    def cplx(a):
        return a.reshape(-1, 2)[:, 0] + 1j * a.reshape(-1, 2)[:, 1]

    def times(z, a):
        q = z * cplx(a)
        return np.stack([q.real, q.imag], -1).reshape(a.shape)

    r = oracle.prepare(DIMS, U, kappa, b) / np.linalg.norm(b)
    v = oracle.mhat(DIMS, U, kappa, r)
    s = r - times(np.vdot(cplx(r), cplx(r)) / np.vdot(cplx(r), cplx(v)), v)
    t = oracle.mhat(DIMS, U, kappa, s)
    e = s - times(np.vdot(cplx(t), cplx(s)) / np.vdot(cplx(t), cplx(t)), t)
    return np.linalg.norm(r), np.linalg.norm(s), np.linalg.norm(e)


def start(kappa, inner, **kw):
    U = wdinputs.gauge_random(DIMS, 0.3, 5)
    s = Setup(DIMS, U, precs=tuple({"fp64", inner}))
    bs = wdinputs.spinor_gaussian(DIMS, 60, nrhs=NRHS)
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    params = wd.solve_params(tol=1e-13, maxiter=1, inner=inner, nrhs=NRHS, **kw)
    ws = wd.new_workspace(s.lat, params, "bicgstab")
    return U, bs, s, wd.Solver("bicgstab", s.gauge, kappa, torch.zeros_like(bt), bt, params, ws)


@pytest.mark.parametrize("inner,unit", [("fp64", 2.0 ** -53), ("fp32", 2.0 ** -24)])
def test_residual_norm_of_a_steep_step(inner, unit):
    kappa = 0.007
    U, bs, _, h = start(kappa, inner, delta=0.0)
    h.step(1)
    got = [q[0] for q in h.residuals()]
    h.end()
    for k in range(NRHS):
        r0, s, r = one_step(U, kappa, bs[k])
        assert 5e-4 < s / r0 < 2e-3 and 5e-4 < r / s < 2e-3
        bound = 8 * unit * (r0 / s + s / r) * (2 if inner == "fp64" else 1)
        assert abs(got[k] / r ** 2 - 1) <= bound, k


@pytest.mark.parametrize("inner", ["fp64", "fp32", "i16", "f16"])
@pytest.mark.parametrize("restart,delta", [(False, 0.0), (True, 1e-9)])
def test_a_steep_step_brings_no_update_of_its_own(inner, restart, delta):
    """|r| falls to 4e-8 |r0| and to 2e-4 |s|: above tol, and above delta |r0|."""
    _, _, _, h = start(0.003, inner, delta=delta, restart=restart)
    h.step(1)
    st, infos = h.end()
    assert st == wd.WD_NOT_CONVERGED
    assert [(i["iters"], i["reliable_updates"]) for i in infos] == [(1, 0)] * NRHS


@pytest.mark.parametrize("solver", ["bicgstab", "cg"])
@pytest.mark.parametrize("inner", ["fp32", "f16"])
def test_step_reports_an_update_that_converges(solver, inner):
    """tol just above the true residual of a reliable update: the step that ran it
    is the one that reports done, also where the iterated residual was still
    above tol."""
    dims, kappa = (6, 4, 6, 10), 0.124
    s = Setup(dims, wdinputs.gauge_random(dims, 0.3, 7), precs=("fp64", inner))
    bt = torch.from_numpy(np.ascontiguousarray(wdinputs.spinor_gaussian(dims, 8, nrhs=1))).to(DEV)

    def steps(tol, most):
        """(done, relative true residual at the last update) after each step."""
        params = wd.solve_params(tol=tol, maxiter=2000, inner=inner, delta=0.1)
        h = wd.Solver(solver, s.gauge, kappa, torch.zeros_like(bt), bt, params, wd.new_workspace(s.lat, params, solver))
        out = []
        while len(out) < most and not (out and out[-1][0]):
            done = h.step(1)
            q = h.residuals()[0]
            out.append((done, float(np.sqrt(q[1] / q[2]))))
        h.end()
        return out

    ref = steps(1e-13, 2000)
    assert ref[-1][0]
    best, tried = ref[0][1], 0
    for k in range(1, len(ref)):
        if ref[k][1] >= best:
            continue
        best = ref[k][1]
        got = steps(best * (1 + 1e-12), k + 4)
        assert [d for d, _ in got] == [False] * k + [True], k
        tried += 1
    assert tried >= 5
