"""Kernels that move tiles through LDS, streaming stores, and the sizes at which
the solvers change their launches.

Tiles hold 64 sites of a parity (spinors) or of the lattice (links): lattices
below one tile, with a remainder of 8 or 16 sites, and of several tiles.
Bounds: conversions to FP64 are exact and to FP32 one rounding; the 16-bit
formats and the operators keep the bars of the other tests; 3x3 products of
links of modulus <= 1 stay within 1e-12 over a temporal extent of 6."""
import numpy as np
import pytest

import oracle
import paper_0911_3191_amd as wd
import wdinputs
from gpu_helpers import DEV, Setup, rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DIMS = [(2, 2, 4, 2), (6, 2, 2, 6), (2, 6, 10, 4)]
TOL = {"fp64": 1e-13, "fp32": 1e-6, "i16": 2e-3, "f16": 2e-3}


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", ["fp64", "fp32", "i16", "f16"])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_spinor_conversions_of_partial_tiles(dims, prec, nrhs):
    s = Setup(dims, wdinputs.gauge_random(dims, 0.3, 91), precs=(prec,))
    psi = wdinputs.spinor_gaussian(dims, 92, nrhs=nrhs).reshape((nrhs,) + tuple(dims[::-1]) + (4, 3, 2))
    halves = [np.stack([oracle.split(dims, psi[k])[p] for k in range(nrhs)]) for p in (0, 1)]
    back = torch.full((psi.size,), 7.0, dtype=torch.float64, device=DEV)
    for p in (0, 1):
        f = s.encode_full(prec, psi, p, nrhs)
        one = s.decode(prec, f, nrhs).reshape(nrhs, -1)
        want = halves[p].reshape(nrhs, -1)
        if prec == "fp64":
            assert np.array_equal(one, want)
        elif prec == "fp32":
            assert np.array_equal(one, want.astype(np.float32).astype(np.float64))
        else:
            assert rel_l2(one, want) <= TOL[prec]
        # the parity array gives the same field; a basis change and back the same values
        assert np.array_equal(s.decode(prec, s.encode_parity(prec, halves[p], nrhs), nrhs).reshape(nrhs, -1), one)
        uk = s.decode(prec, s.encode_parity(prec, halves[p], nrhs, basis=1), nrhs, basis=1)
        assert rel_l2(uk.reshape(nrhs, -1), want) <= max(TOL[prec], 1e-15)
        before = back.clone()
        wd.wd_spinor_decode_full(s.lat, prec, nrhs, p, back, f)
        torch.cuda.synchronize()
        now = back.cpu().numpy().reshape(psi.shape)
        old = before.cpu().numpy().reshape(psi.shape)
        for k in range(nrhs):
            got = oracle.split(dims, now[k])
            assert np.array_equal(np.ravel(got[p]), one[k])
            assert np.array_equal(got[1 - p], oracle.split(dims, old[k])[1 - p])  # the other parity is not touched


@pytest.mark.parametrize("dims", DIMS)
def test_gauge_setup_of_partial_tiles(dims):
    U = wdinputs.gauge_random(dims, 0.5, 93)
    lat = wd.lattice(dims)
    Uf, g = wd.gauge_fix_temporal(lat, torch.from_numpy(U).to(DEV))
    Uo, go = oracle.gauge_fix_temporal(dims, U)
    assert np.abs(Uf.cpu().numpy().reshape(Uo.shape) - Uo).max() < 1e-12
    psi = wdinputs.spinor_gaussian(dims, 94, nrhs=3)
    pd = torch.from_numpy(psi).to(DEV)
    out = torch.empty_like(pd)
    wd.wd_gauge_rotate_spinor(lat, g, out, pd, 3)
    torch.cuda.synchronize()
    ref = oracle.gauge_rotate_spinor(dims, go, psi)
    assert np.abs(out.cpu().numpy().reshape(ref.shape) - ref).max() < 1e-12
    for prec in TOL:
        for recon, links, temporal in ((12, U, False), (8, U, False), (12, Uo, True), (8, Uo, True)):
            s = Setup(dims, links, precs=(prec,), recon=recon, temporal=temporal)
            for p in (0, 1):
                src = oracle.split(dims, psi[0])[1 - p]
                f, o = s.encode_parity(prec, src[None]), s.field(prec)
                wd.wd_dslash_field(s.gauge, o, f, p, 0, prec, 1)
                assert rel_l2(s.decode(prec, o), oracle.dslash_parity(dims, links, src, p)) <= TOL[prec], (prec, recon)


@pytest.mark.parametrize("dims", [(6, 10, 16, 4), (10, 6, 6, 12)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "i16", "f16"])
def test_streaming_stores_keep_the_bits(prec, dims, monkeypatch):
    """Field 5 of the shape: the dslash stores its output past the caches."""
    nrhs, kappa = 5, 0.122
    U = wdinputs.gauge_random(dims, 0.3, 95)
    s = Setup(dims, U, precs=tuple({"fp64", prec}))
    bs = wdinputs.spinor_gaussian(dims, 96, nrhs=nrhs)
    pe = np.stack([oracle.split(dims, b)[0] for b in bs])
    fin = s.encode_parity(prec, pe, nrhs, basis=0)
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    params = wd.solve_params(tol=1e-10, inner=prec, delta=0.0 if prec == "fp64" else 0.1, nrhs=nrhs)
    shapes = [f"{nr},0,1,0,%d" for nr in (1, 2, 3)] + ["1,0,1,0,%d,0,0,0,256,1"]
    if prec == "f16":
        shapes += ["1,0,1,0,%d,0,0,1", "1,0,1,0,%d,0,1,1"]
    ref = None
    for shape in shapes:
        for nt in (0, 1):
            monkeypatch.setenv("WD_DSLASH_SHAPE", shape % nt)
            tmp, m = s.field(prec, nrhs), s.field(prec, nrhs)
            wd.wd_mat_pc_field(s.gauge, kappa, m, fin, tmp, 0, prec, nrhs)
            got = [s.decode(prec, tmp, nrhs), s.decode(prec, m, nrhs)]
            for solver, fn in (("bicgstab", wd.bicgstab_solve), ("cg", wd.cg_solve)):
                x = torch.zeros_like(bt)
                fn(s.gauge, kappa, x, bt, params, wd.new_workspace(s.lat, params, solver))
                torch.cuda.synchronize()
                got.append(x.cpu().numpy())
            ref = ref or got
            for a, b in zip(got, ref):
                assert np.array_equal(a, b), (shape, nt)
    for k in range(nrhs):
        assert rel_l2(ref[1][k], oracle.mhat(dims, U, kappa, pe[k])) <= TOL[prec]
        for x in ref[2:]:
            assert oracle.true_relres(dims, U, kappa, bs[k], x[k]) <= 1e-10


# 32,768 sites of a parity are the most that finish a dot in its own launch,
# 65,536 the most whose FP64 and FP32 updates split a site over threads.
@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (12, 10, 20, 28), (16, 16, 16, 32), (12, 16, 24, 30)])
@pytest.mark.parametrize("solver", ["bicgstab", "cg"])
@pytest.mark.parametrize("inner", ["fp64", "fp32", "f16"])
def test_solves_on_both_sides_of_the_launch_rules(dims, solver, inner, monkeypatch):
    nrhs, kappa = 2, 0.12
    U = wdinputs.gauge_random(dims, 0.3, 97)
    s = Setup(dims, U, precs=tuple({"fp64", inner}))
    bs = wdinputs.spinor_gaussian(dims, 98, nrhs=nrhs)
    bt = torch.from_numpy(np.ascontiguousarray(bs)).to(DEV)
    fn = wd.bicgstab_solve if solver == "bicgstab" else wd.cg_solve
    ref = None
    for every, graph, shape in ((1, False, None), (5, True, None), (2, False, "1,0,1"),
                                (2, False, "1,0,1,0,0,0,0,0,256,1")):
        if shape:  # block records and wave records
            monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
        params = wd.solve_params(tol=1e-10, inner=inner, delta=0.0 if inner == "fp64" else 0.1, nrhs=nrhs,
                                 use_graph=graph, check_every=every)
        x = torch.zeros_like(bt)
        st, infos = fn(s.gauge, kappa, x, bt, params, wd.new_workspace(s.lat, params, solver), torch.cuda.Stream())
        torch.cuda.synchronize()
        assert st == wd.WD_OK
        got = (x.cpu().numpy(), [(i["iters"], i["reliable_updates"]) for i in infos])
        ref = ref or got
        assert got[1] == ref[1]
        assert np.array_equal(got[0], ref[0])
    for k in range(nrhs):
        assert oracle.true_relres(dims, U, kappa, bs[k], ref[0][k]) <= 1e-10


@pytest.mark.parametrize("inner", ["fp64", "f16"])
def test_a_step_that_solves_the_system_ends_it(inner):
    """kappa 1e-14: M_hat rounds to 1, so the first step leaves s = 0 and omega,
    rho, beta and |r| come from zero dots."""
    dims = (4, 4, 4, 6)
    s = Setup(dims, wdinputs.gauge_random(dims, 0.3, 99), precs=tuple({"fp64", inner}))
    b = torch.from_numpy(np.ascontiguousarray(wdinputs.spinor_gaussian(dims, 100, nrhs=1))).to(DEV)
    x, info = wd.solve_full("bicgstab", s.gauge, s.lat, 1e-14, b, tol=1e-12, inner=inner,
                            delta=0.0 if inner == "fp64" else 0.1)
    assert info["converged"] == 1
    # |x - b| <= |r| + |kappa D x| <= (tol + 8 kappa) |b|
    assert rel_l2(x.cpu().numpy(), b.cpu().numpy()) <= 1.1e-12
