"""The register line FFT (N = 64, 128, 256) where the other spectrum and jump
tests do not reach it: the remaining combinations of size, precision and
number of fields."""
import numpy as np
import pytest

import workloads as W
from test_gpu_spectrum import check

pytestmark = pytest.mark.gpu


def _lib():
    from paper_2607_24978_amd import _lib
    return _lib


@pytest.mark.parametrize("N,precision", [(64, "fp64"), (128, "fp32"), (256, "fp64")])
def test_spectrum_sizes(N, precision):
    """pi of a noise state (rows are transformed in pairs) against the numpy DFT."""
    f, p = W.random_state(N, 1, 5)
    lat = _lib().Lattice(N, 0.2, 1, precision)
    lat.set_background(1.0, "static", 1.0, 1.0)
    lat.set_fields(f, p)
    _, pd = lat.get_fields()
    check(lat, pd[0], 0, "pi", 1.0, 0.2)
    lat.close()


@pytest.mark.parametrize("nf,N", [(1, 64), (2, 64), (1, 128), (2, 128), (1, 256)])
def test_linear_jump_fp32_sizes(nf, N):
    """One linear jump of an FP32 lattice, whose x transforms run with the
    modes at these sizes, against the oracle's FP64 jump from the same state:
    allowed 4 eps32 of the values and 64 eps32 of the fluctuations, the bound
    of the FP32 transforms (2 log2(N^3) stages of a few eps32)."""
    from oracle import lattice as L
    from oracle import propagator as PR
    lib = _lib()
    w = W.C1.with_(N=N, k_ir=1.0 * 32 / N, precision="fp32")
    g2 = 3.0 if nf == 2 else 0.0
    P = L.Params(N=N, dx=w.dx, n_fields=nf, m2=(0.0, 0.0), lam=w.lam, g2=g2, V0=0.0)
    f, p = W.random_state(N, nf, 9, famp=1e-3, pamp=1e-3)
    f, p = f.astype(np.float32).astype(np.float64), p.astype(np.float32).astype(np.float64)
    rho, _ = L.rho_pressure(*L.energies(f, p, 1.0, P))
    s0 = L.State(f, p, 1.0, L.hubble_from_rho(1.0, rho, P))
    lat = lib.Lattice(N, w.dx, nf, "fp32")
    lat.set_potential((0.0, 0.0), w.lam, g2, 0.0)
    lat.set_fields(f, p)
    sg = lib.Surrogate(n_fields=nf, extra_inputs=2, layers=2, jump_steps=4, init_seed=1)
    sg.set_jump("linear")
    sg.set_gate(0.0)
    _, rep = sg.advance(lat, "leapfrog", w.dt, 1, threshold=float("inf"))
    assert rep["fallbacks"] == 0
    got = lat.get_fields()
    s, _ = PR.linear_jump(s0, w.dt, 4, "leapfrog", P)
    eps = float(np.finfo(np.float32).eps)
    for g, want in zip(got, (s.f, s.p)):
        fl = want - want.mean(axis=(1, 2, 3), keepdims=True)
        assert np.max(np.abs(g - want)) <= 4 * eps * np.max(np.abs(want)) + 64 * eps * np.max(np.abs(fl))
    lat.close()
    sg.close()
