"""The rules that choose a pass's tile, called in the built library on the CPU
(they take sizes only): every lattice size that cl_create accepts."""
import ctypes as C

import pytest

PREC = {"fp64": 0, "fp32": 1}
MAX_BLOCKS = 4096   # workgroups of a pass whose partial sums the next one reads
TUNED_BLOCKS = 1024


class Tile(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("TZ", "TY", "CX", "RY", "NT", "HI", "PD", "nbz", "nby", "nbx")]

    @property
    def nblocks(self):
        return self.nbz * self.nby * self.nbx

    def fits(self, N):
        return (self.nbz * self.TZ == N and self.nby * self.TY == N and self.nbx * self.CX == N
                and self.NT <= 512 and self.nblocks <= MAX_BLOCKS)

    def __str__(self):
        return str([getattr(self, k) for k, _ in self._fields_])


def rule(name, restype, *argtypes):
    from paper_2607_24978_amd import _lib
    f = getattr(C.CDLL(_lib.LIB_PATH), name)
    f.restype, f.argtypes = restype, argtypes
    return f


def default_tile(N, prec, nf):
    return rule("_ZN2cl12default_tileEi12cl_precisioni", Tile, C.c_int, C.c_int, C.c_int)(N, PREC[prec], nf)


def reduction_tile(t, N, prec, nf):
    f = rule("_ZN2cl14reduction_tileERKNS_4TileEi12cl_precisioni", Tile, C.POINTER(Tile), C.c_int, C.c_int, C.c_int)
    return f(C.byref(t), N, PREC[prec], nf)


def candidates(N, prec, nf):
    f = rule("_ZN2cl15candidate_tilesEi12cl_precisioniPNS_4TileEPii", None, C.c_int, C.c_int, C.c_int, C.POINTER(Tile),
             C.POINTER(C.c_int), C.c_int)
    out, n = (Tile * 1024)(), C.c_int()
    f(N, PREC[prec], nf, out, C.byref(n), len(out))
    return list(out[:n.value])


def sizes(prec):
    big = 256 if prec == "fp32" else 128
    return [N for N in range(8, 1601, 2) if N & (N - 1) == 0 or N % big == 0]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nf", [1, 2])
def test_reductions_fit(prec, nf):
    """The reductions of a lattice in its default tile or in any tile the
    autotuner may pick are valid tiles of at most TUNED_BLOCKS workgroups, or
    of as many as the tile itself."""
    for N in sizes(prec):
        for t in [default_tile(N, prec, nf)] + candidates(N, prec, nf):
            assert t.fits(N), (N, str(t))
            r = reduction_tile(t, N, prec, nf)
            assert r.fits(N) and r.NT == t.NT, (N, str(t), str(r))
            assert r.nblocks <= max(t.nblocks, TUNED_BLOCKS), (N, str(t), str(r))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nf", [1, 2])
def test_reduction_march_and_depth(prec, nf):
    """A reduction keeps the march of a tile with more workgroups than CUs, and
    of two fields in eight-wave workgroups; of one field, eight-wave workgroups
    that are more than the CUs run at depth 1."""
    seen = set()
    for N in sizes(prec):
        for t in [default_tile(N, prec, nf)] + candidates(N, prec, nf):
            r = reduction_tile(t, N, prec, nf)
            wide = t.NT > 256
            if t.nblocks > 256 or (wide and nf == 2):
                assert r.CX == t.CX, (N, str(t))
                seen.add("march")
            if wide and nf == 1 and r.nblocks > 256:
                assert r.PD == 1, (N, str(t))
                seen.add("depth")
    assert seen == ({"march", "depth"} if nf == 1 else {"march"})


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_waves_tile(prec):
    """The tile with the gravitational-wave tensor is valid at every size (those
    whose state fits the memory: at most 1024), and where its columns alone
    occupy the chip the marches still make at least two rounds of workgroups."""
    f = rule("_ZN2cl7gw_tileEi12cl_precision", Tile, C.c_int, C.c_int)
    for N in sizes(prec):
        if N > 1024:
            continue
        t = f(N, PREC[prec])
        assert t.fits(N) and t.NT <= 256 and (t.RY, t.PD) == (1, 1), (N, str(t))
        if t.nbz * t.nby >= 512:
            assert t.nblocks >= 1024, (N, str(t))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_default_march_of_one_field(prec):
    """Two four-wave workgroups of one field run on a CU: from 128^3 on their
    march gives the chip 512 of them, as far as the lattice has columns for."""
    seen = 0
    for N in sizes(prec):
        t = default_tile(N, prec, 1)
        if N >= 128 and t.NT == 256:
            seen += 1
            assert t.nblocks >= 512, (N, str(t))
    assert seen
