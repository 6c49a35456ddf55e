"""Default tiles and the march direction of the lattice passes.

Odd passes of a call march their tiles' planes downwards, and the default tile follows the size of the lattice (one to eight
waves per workgroup, marches from one plane up).  In static space the fields
do not depend on the lattice sums, and the site update rounds the same in
every tile and direction: a run in the default tile equals one in another
tile bitwise, and the sums agree to the rounding of their summation order
(FP64: 4 eps per level of a sum over 2^k terms is below 1e-12; FP32 lattices
round each thread's plane partials to FP32, 1e-6 as bounded for their sums).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _run(N, nf, precision, tile, integrator, n):
    from paper_2607_24978_amd import _lib as lib
    f, p = W.random_state(N, nf, 7)
    lat = lib.Lattice(N, 0.5, nf, precision)
    if tile:
        lat.set_tile(*tile)
    lat.set_background(expansion="static")
    lat.set_potential(lam=(1.0, 0.5), g2=2.0 if nf == 2 else 0.0)
    lat.set_fields(f, p)
    r = lat.step(integrator, 0.02, n)
    out = lat.get_fields()
    used = lat.get_tile()
    lat.close()
    return r, out, used


@pytest.mark.parametrize("N,nf,precision,tile", [
    (8, 1, "fp64", (8, 4, 8)),       # 32-thread default, marches of one plane
    (16, 2, "fp32", (16, 8, 16)),    # one wave, one plane
    (32, 1, "fp64", (32, 16, 8)),
    (64, 2, "fp32", (32, 16, 64)),   # two waves, two planes
    (128, 1, "fp32", (64, 16, 32)),  # four waves
    (128, 2, "fp64", (32, 8, 128)),  # four waves, streaming stores start above this size
    (256, 2, "fp64", (64, 4, 128)),  # eight waves, streaming stores
    (384, 1, "fp64", (64, 8, 384)),  # eight waves, an odd number of chunks
])
@pytest.mark.parametrize("integrator", ["leapfrog", "rk3"])
def test_default_tile_equals_another(N, nf, precision, tile, integrator):
    if integrator == "rk3" and N > 128:
        pytest.skip("the stage pass shares the march, covered at the smaller sizes")
    a = _run(N, nf, precision, None, integrator, 2)
    b = _run(N, nf, precision, tile, integrator, 2)
    assert (a[2]["tz"], a[2]["ty"], a[2]["cx"]) != tile
    assert np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
    tol = 1e-12 if precision == "fp64" else 1e-6
    for k in ("EK", "EG", "EV", "var"):
        assert np.all(np.abs(a[0][k] - b[0][k]) <= tol * np.abs(b[0][k])), k
