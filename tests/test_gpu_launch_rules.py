"""Solves long enough to be captured, and lattices at the sizes where a solver's
launches change."""
import numpy as np
import pytest

import oracle
import paper_0911_3191_amd as wd
import wdinputs
from gpu_helpers import DEV, Setup

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SLOT, SPLIT = "1,0,1", "1,0,1,0,0,0,0,0,256,1"


def solve(s, solver, bt, kappa, **kw):
    params = wd.solve_params(nrhs=bt.shape[0], maxiter=4000, **kw)
    x = torch.zeros_like(bt)
    fn = wd.bicgstab_solve if solver == "bicgstab" else wd.cg_solve
    torch.cuda.synchronize()
    st, infos = fn(s.gauge, kappa, x, bt, params, wd.new_workspace(s.lat, params, solver), torch.cuda.Stream())
    torch.cuda.synchronize()
    assert st == wd.WD_OK, infos
    return x.cpu().numpy(), [(i["iters"], i["reliable_updates"]) for i in infos]


@pytest.mark.parametrize("solver,inner,restart", [("bicgstab", "fp64", False), ("bicgstab", "fp32", False),
                                                  ("bicgstab", "f16", False), ("bicgstab", "f16", True),
                                                  ("cg", "fp64", False), ("cg", "f16", False)])
@pytest.mark.parametrize("shape", [SLOT, SPLIT])
def test_captured_batches_give_the_bits_of_direct_launches(solver, inner, restart, shape, monkeypatch):
    """With use_graph a solve is captured after 12 batches of check_every
    iterations; two iterations a batch, each its own place in it."""
    dims, kappa = (8, 4, 8, 6), 0.14
    U = wdinputs.gauge_random(dims, 0.4, 13)
    s = Setup(dims, U, precs=tuple({"fp64", inner}))
    bs = wdinputs.spinor_gaussian(dims, 14, nrhs=3)
    bs[1] = 0.0
    bs[1][0, 0, 0, 0, 2, 1, 0] = 1.0  # updates of part of the batch
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
    kw = dict(tol=1e-12, inner=inner, delta=0.0 if inner == "fp64" else 0.1, restart=restart)
    x0, n0 = solve(s, solver, bt, kappa, use_graph=False, check_every=1, **kw)
    x1, n1 = solve(s, solver, bt, kappa, use_graph=True, check_every=2, **kw)
    assert max(k - l for k, l in n1) >= 2 * 14, n1  # at least 14 batches: the last two or more are replays
    assert n1 == n0
    assert np.array_equal(x1, x0)
    for k in range(3):
        assert oracle.true_relres(dims, U, kappa, bs[k], x1[k]) <= 1e-12


# A launch finishes its own dot up to 128 records: 8,192 sites of a parity for a
# split dslash (one record per 64 sites; z slabs or a contiguous range) and for
# the FP64 x/r update, 16,384 for the FP32 one, 32,768 for the 16-bit one.
@pytest.mark.parametrize("dims", [(16, 16, 8, 8), (16, 16, 4, 16), (16, 16, 8, 10), (12, 20, 6, 12),
                                  (16, 16, 16, 8), (16, 16, 16, 10)])
@pytest.mark.parametrize("solver", ["bicgstab", "cg"])
@pytest.mark.parametrize("inner", ["fp64", "fp32", "f16"])
def test_solves_at_the_largest_fused_finalize(dims, solver, inner, monkeypatch):
    kappa = 0.12
    U = wdinputs.gauge_random(dims, 0.3, 117)
    s = Setup(dims, U, precs=tuple({"fp64", inner}))
    bs = wdinputs.spinor_gaussian(dims, 118, nrhs=2)
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    ref = None
    for every, shape in ((1, SLOT), (3, SPLIT), (1, None)):
        if shape:
            monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
        else:
            monkeypatch.delenv("WD_DSLASH_SHAPE")
        got = solve(s, solver, bt, kappa, tol=1e-10, inner=inner, delta=0.0 if inner == "fp64" else 0.1,
                    check_every=every)
        ref = ref or got
        assert got[1] == ref[1]
        assert np.array_equal(got[0], ref[0])
    for k in range(2):
        assert oracle.true_relres(dims, U, kappa, bs[k], ref[0][k]) <= 1e-10
