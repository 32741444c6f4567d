"""One-thread launch shapes on the link formats, forced: small lattices take the
split kernel by themselves, large ones these.

8-real links have kernels of one and two slots; links in temporal gauge (unit
links off the last time slice) run under 1-4 slots, LDS staging (16-bit formats,
Lz a multiple of 8) and the binary16 RHS loop.  Every shape redistributes the
same arithmetic: the bits of each right-hand side alone, and the oracle's values
within the bars of the other tests."""
import numpy as np
import pytest

import oracle
import paper_0911_3191_amd as wd
import wdinputs
from gpu_helpers import Setup, rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {"fp64": 1e-13, "fp32": 1e-6, "i16": 2e-3, "f16": 2e-3}
SLOT = "1,0,1"


def check_shapes(s, links, dims, prec, nrhs, shapes, monkeypatch):
    src = wdinputs.spinor_gaussian(dims, 112, nrhs=nrhs)
    po = np.stack([oracle.split(dims, src[k])[1] for k in range(nrhs)])
    for basis in (0, 1):
        fin = s.encode_parity(prec, po, nrhs, basis=basis)
        for dagger in (0, 1):
            monkeypatch.setenv("WD_DSLASH_SHAPE", SLOT)
            alone = []
            for k in range(nrhs):
                f1, o1 = s.encode_parity(prec, po[k:k + 1], basis=basis), s.field(prec)
                wd.wd_dslash_field_basis(s.gauge, o1, f1, 0, dagger, prec, 1, basis)
                alone.append(s.decode(prec, o1, basis=basis))
                ref = oracle.dslash_parity(dims, links, po[k], 0, dagger=bool(dagger))
                assert rel_l2(alone[k], ref) <= TOL[prec], (basis, dagger, k)
            for shape in shapes:
                monkeypatch.setenv("WD_DSLASH_SHAPE", shape)
                out = s.field(prec, nrhs)
                wd.wd_dslash_field_basis(s.gauge, out, fin, 0, dagger, prec, nrhs, basis)
                assert np.array_equal(s.decode(prec, out, nrhs, basis=basis), np.stack(alone)), (shape, basis, dagger)


@pytest.mark.parametrize("dims", [(4, 6, 8, 4), (6, 4, 6, 10)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "i16", "f16"])
@pytest.mark.parametrize("temporal", [False, True])
def test_recon8_slots(prec, dims, temporal, monkeypatch):
    U = wdinputs.gauge_random(dims, 0.5, 111)
    links = oracle.gauge_fix_temporal(dims, U)[0] if temporal else U
    s = Setup(dims, links, precs=(prec,), recon=8, temporal=temporal)
    check_shapes(s, links, dims, prec, 3, [SLOT, "2,0,1", "2,1,2", "2,0,1,0,0,0,0,0,128"], monkeypatch)


@pytest.mark.parametrize("dims", [(6, 4, 8, 6), (4, 6, 6, 4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "i16", "f16"])
def test_temporal_gauge_shapes(prec, dims, monkeypatch):
    U = wdinputs.gauge_random(dims, 0.5, 113)
    links = oracle.gauge_fix_temporal(dims, U)[0]
    s = Setup(dims, links, precs=(prec,), recon=12, temporal=True)
    shapes = [f"{nr},0,1" for nr in (1, 2, 3, 4)]
    slab = dims[2] % 8 == 0
    if prec in ("i16", "f16") and slab:
        shapes += [f"{nr},0,1,0,0,0,1" for nr in (1, 2, 3)]
    if prec == "f16":
        shapes += ["1,0,1,0,0,0,0,1"] + (["1,0,1,0,0,0,1,1"] if slab else [])
    check_shapes(s, links, dims, prec, 5, shapes, monkeypatch)


def test_the_recorded_shape_gives_the_bits_of_the_launch(tmp_path, monkeypatch):
    """The tuner records the best one-thread shape of a key whose launches take
    the split kernel; forced, it gives the same bits."""
    dims, nrhs, prec = (6, 12, 16, 4), 3, "f16"  # a lattice no other test launches
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("WD_TUNE_CACHE", str(cache))
    monkeypatch.delenv("WD_TUNE", raising=False)
    monkeypatch.delenv("WD_DSLASH_SHAPE", raising=False)
    U = wdinputs.gauge_random(dims, 0.4, 114)
    s = Setup(dims, U, precs=(prec,))
    src = wdinputs.spinor_gaussian(dims, 115, nrhs=nrhs)
    po = np.stack([oracle.split(dims, src[k])[1] for k in range(nrhs)])
    fin = s.encode_parity(prec, po, nrhs, basis=1)

    def run():
        out = s.field(prec, nrhs)
        wd.wd_dslash_field_basis(s.gauge, out, fin, 0, 0, prec, nrhs, 1)
        return s.decode(prec, out, nrhs, basis=1)

    first = run()
    lines = cache.read_text().splitlines()
    assert len(lines) == 1
    nr, block, gslow, nsub, nt, lds, rloop, wgs = [int(v) for v in lines[0].split()][8:]
    monkeypatch.setenv("WD_DSLASH_SHAPE", f"{nr},{gslow},{nsub},{nt & 1},{nt >> 1},{wgs},{lds},{rloop},{block},0")
    assert np.array_equal(run(), first)
    for k in range(nrhs):
        assert rel_l2(first[k], oracle.dslash_parity(dims, U, po[k], 0)) <= TOL[prec]
