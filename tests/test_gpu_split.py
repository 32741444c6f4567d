"""The one-wavefront-per-hop dslash gives the bits of the one-thread kernels.

Forced launch shapes: "1,0,1" is the one-slot kernel, SPLIT the split one.
Lattices: fewer sites than one workgroup, z slabs whose last workgroup is not
full (Lz a multiple of 8), a contiguous range (Lz not a multiple of 8).  The
solvers run every fused dot product, the FP64 residual and its re-encoding."""
import numpy as np
import pytest

import oracle
import paper_0911_3191_amd as wd
import wdinputs
from gpu_helpers import DEV, Setup, rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SLOT, SPLIT = "1,0,1", "1,0,1,0,0,0,0,0,256,1"
TOL = {"fp64": 1e-13, "fp32": 1e-6, "i16": 2e-3, "f16": 2e-3}


@pytest.mark.parametrize("dims", [(2, 2, 4, 2), (6, 10, 16, 4), (10, 6, 6, 12)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "i16", "f16"])
def test_split_operators_give_the_one_thread_bits(prec, dims, monkeypatch):
    nrhs, kappa = 3, 0.124
    U = wdinputs.gauge_random(dims, 0.3, 81)
    Ut = oracle.gauge_fix_temporal(dims, U)[0]
    srcs = wdinputs.spinor_gaussian(dims, 82, nrhs=nrhs)
    po = np.stack([oracle.split(dims, srcs[k])[1] for k in range(nrhs)])
    for recon, temporal in ((12, False), (8, True)):
        links = Ut if temporal else U
        s = Setup(dims, links, precs=(prec,), recon=recon, temporal=temporal)
        for basis in (0, 1):
            fin = s.encode_parity(prec, po, nrhs, basis=basis)
            for dagger in (0, 1):
                got = []
                for shape in (SLOT, SPLIT):
                    monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
                    f = s.field(prec, nrhs)
                    wd.wd_dslash_field_basis(s.gauge, f, fin, 0, dagger, prec, nrhs, basis)
                    got.append(s.decode(prec, f, nrhs, basis=basis))
                    if basis == 0:
                        tmp, m = s.field(prec, nrhs), s.field(prec, nrhs)
                        wd.wd_mat_pc_field(s.gauge, kappa, m, f, tmp, dagger, prec, nrhs)
                        got[-1] = (got[-1], s.decode(prec, m, nrhs))
                assert np.array_equal(got[0], got[1]), (recon, basis, dagger)
                first = got[1] if basis else got[1][0]
                for k in range(nrhs):
                    ref = oracle.dslash_parity(dims, links, po[k], 0, dagger=bool(dagger))
                    assert rel_l2(first[k], ref) <= TOL[prec], (recon, basis, dagger, k)


@pytest.mark.parametrize("solver,restart", [("bicgstab", False), ("cg", False), ("bicgstab", True)])
@pytest.mark.parametrize("inner", ["fp64", "fp32", "i16", "f16"])
def test_split_solves_give_the_one_thread_bits(solver, restart, inner, monkeypatch):
    if restart and inner == "fp64":
        pytest.skip("defect correction runs a lower inner precision")
    dims, kappa, nrhs = (6, 10, 8, 4), 0.122, 3
    U = wdinputs.gauge_random(dims, 0.3, 83)
    s = Setup(dims, U, precs=tuple({"fp64", inner}))
    bs = wdinputs.spinor_gaussian(dims, 84, nrhs=nrhs)
    bs[1] = 0.0
    bs[1][0, 0, 0, 0, 2, 1, 0] = 1.0  # converges on its own schedule: updates of part of the batch
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    params = wd.solve_params(tol=1e-12, inner=inner, delta=0.0 if inner == "fp64" else 0.1, nrhs=nrhs,
                             use_graph=True, restart=restart)
    got = []
    for shape in (SLOT, SPLIT):
        monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
        ws = wd.new_workspace(s.lat, params, solver)
        x = torch.zeros_like(bt)
        fn = wd.bicgstab_solve if solver == "bicgstab" else wd.cg_solve
        torch.cuda.synchronize()
        st, infos = fn(s.gauge, kappa, x, bt, params, ws, torch.cuda.Stream())
        assert st == wd.WD_OK, infos
        got.append((x.cpu().numpy(), [(i["iters"], i["reliable_updates"]) for i in infos]))
    assert got[0][1] == got[1][1]
    assert np.array_equal(got[0][0], got[1][0])
    for k in range(nrhs):
        assert oracle.true_relres(dims, U, kappa, bs[k], got[1][0][k]) <= 1e-12
