"""GPU parity of the gravitational-wave tensor (five traceless components
carried in the fused pass, Sect. 4.2) against the CPU FP64 oracle, through
the C ABI.  FP64: tensor fields within 1e-11 (norm-wise) of the oracle and the
scalar records unchanged at 1e-11; FP32: a bound derived from the storage
rounding of the fields that source the tensor."""
import math

import numpy as np
import pytest

from oracle import gw as G
from oracle import lattice as L
import workloads as W
from test_gpu_parity import compare_records, make_lattice, oracle_seed, params

pytestmark = pytest.mark.gpu


def _lib():
    from paper_2607_24978_amd import _lib
    return _lib


def run_gw_both(w, n, integrator, amp, precision=None, expansion="self"):
    s0 = oracle_seed(w, expansion, amp)
    P = params(w, expansion)
    lat = make_lattice(w, precision=precision, expansion=expansion)
    lat.gw_enable(True)
    lat.set_fields(s0.f, s0.p)
    recs = lat.step(integrator, w.dt, n)
    v, u = lat.gw_get()
    f, p = lat.get_fields()
    st = lat.get_state()
    spec = lat.gw_spectrum()
    lat.close()
    z = np.zeros((5,) + s0.f.shape[1:])
    s, vo, uo = s0, z.copy(), z.copy()
    orecs = []
    for _ in range(n):
        s, vo, uo = G.step(s, vo, uo, w.dt, P, integrator)
        orecs.append(L.observe(s, P))
    return dict(recs=recs, orecs=orecs, v=v, u=u, f=f, p=p, st=st, spec=spec, s=s, vo=vo, uo=uo, P=P)


@pytest.mark.parametrize("integrator,n", [("leapfrog", 30), ("vv4", 12)])
@pytest.mark.parametrize("N", [8, 16, 32])
def test_gw_fp64_against_oracle(integrator, n, N):
    """Two-field preheating potential, self-consistent expansion, seeded
    fluctuations (amplitude 20 so that the source is well resolved): the
    tensor and its momenta after n steps, the scalar records, and the
    binned wave spectrum against the oracle."""
    w = W.C1.with_(N=N, k_ir=2.0 * 16 / N, precision="fp64")
    r = run_gw_both(w, n, integrator, amp=20.0)
    compare_records(r["recs"], r["orecs"], 2, 1e-11)
    for got, want in ((r["v"], r["vo"]), (r["u"], r["uo"])):
        assert np.max(np.abs(want)) > 0
        err = np.max(np.abs(got - want)) / np.max(np.abs(want))
        print(f"N={N} {integrator}: tensor rel err {err:.3g}", flush=True)
        assert err <= 1e-11
    counts, rho, omega, tot = r["spec"]
    oc, orho, oom, otot = G.gw_spectrum(r["uo"], r["s"].a, r["P"], rho_tot=sum(L.energies(r["s"].f, r["s"].p, r["s"].a, r["P"])[0])
                                        + sum(L.energies(r["s"].f, r["s"].p, r["s"].a, r["P"])[1])
                                        + L.energies(r["s"].f, r["s"].p, r["s"].a, r["P"])[2], nbins=len(counts))
    assert np.array_equal(counts, oc)
    assert abs(tot - otot) <= 1e-10 * otot
    assert np.max(np.abs(rho - orho)) <= 1e-10 * np.max(orho)
    assert np.max(np.abs(omega - oom)) <= 1e-10 * np.max(np.abs(oom))


def test_gw_fp32_against_oracle():
    """FP32 storage: every stored field carries a rounding of u |f| while the
    source is built from differences of neighbouring values of size |D f|,
    so the tensor is known to about (number of drifts) u max|f| / rms|D f|
    relative; the bar is 20 times that estimate."""
    w = W.C1.with_(N=32, k_ir=1.0, precision="fp32")
    n = 10
    r = run_gw_both(w, n, "leapfrog", amp=20.0, precision="fp32")
    compare_records(r["recs"], r["orecs"], 2, 1e-4, energy_scale=True)
    f = r["s"].f
    dfs = np.sqrt(np.mean([(np.roll(f[j], -1, axis=ax) - f[j]) ** 2 for j in range(2) for ax in range(3)]))
    tol = 20 * (n + 1) * 2.0 ** -24 * np.max(np.abs(f)) / dfs
    for got, want in ((r["v"], r["vo"]), (r["u"], r["uo"])):
        err = np.max(np.abs(got - want)) / np.max(np.abs(want))
        print(f"fp32 tensor rel err {err:.3g} (bar {tol:.3g})", flush=True)
        assert err <= tol < 0.05


@pytest.mark.parametrize("integrator", ["leapfrog", "vv4"])
def test_gw_free_wave_dispersion(integrator):
    """Homogeneous fields source nothing: a cos-mode of v_12 in static space
    follows the massless lattice dispersion (leapfrog cos(n theta), VV4 the
    kick-drift-kick product) to 1e-11."""
    from test_oracle_pins import cos_mode, kdk_matrix, lattice_omega2
    lib = _lib()
    N, dx, nvec = 16, 0.7, (1, 2, 3)
    lat = lib.Lattice(N, dx, 2, "fp64")
    lat.set_background(1.0, "static", 1.0, 1.0)
    lat.set_potential((0.0, 0.0), (1.0, 0.0), 2.0, 0.0)
    lat.gw_enable(True)
    lat.set_fields(np.stack([np.full((N, N, N), 0.8), np.zeros((N, N, N))]), np.zeros((2, N, N, N)))
    g = cos_mode(N, dx, nvec)
    v = np.zeros((5, N, N, N))
    v[1] = 1e-3 * g
    lat.gw_set(v, np.zeros_like(v))
    dt, n = 0.2, 600
    for _ in range(n // 200):
        lat.step(integrator, dt, 200)
    vg, ug = lat.gw_get()
    lat.close()
    w2 = lattice_omega2(N, dx, nvec, 0.0)
    if integrator == "leapfrog":
        M = np.linalg.matrix_power(kdk_matrix(dt, w2), n)
    else:
        M = np.linalg.matrix_power(kdk_matrix(L.W1 * dt, w2) @ kdk_matrix(L.W0 * dt, w2) @ kdk_matrix(L.W1 * dt, w2), n)
    assert np.max(np.abs(vg[1] / 1e-3 - M[0, 0] * g)) <= 1e-11
    assert np.max(np.abs(ug[1] / 1e-3 - M[1, 0] * g)) <= 1e-11 * math.sqrt(w2)
    assert np.max(np.abs(vg[[0, 2, 3, 4]])) == 0.0


@pytest.mark.parametrize("N,nvec,alpha", [(16, (0, 0, 3), 1.0), (16, (1, 2, 3), 1.0), (16, (2, 1, 0), 0.0),
                                          (128, (3, 5, 40), 1.0), (128, (7, 1, 64), 0.0), (128, (64, 3, 20), 1.0)])
def test_gw_spectrum_of_a_prescribed_wave(N, nvec, alpha):
    """A transverse-traceless wave set through the ABI: rho_GW = m_p^2 A^2 /
    (4 a^(2 alpha)) in the bin of |n| (the oracle's pin), and the device
    spectrum equals the oracle's on the same input.  At 128^3 the transforms
    are held for z <= N / 2 only (80 stored z per line): a wave with
    0 < z < N / 2 is counted through its mirror, one at z = N / 2 once, and
    one with x = N / 2 has a mirror whose lattice momentum is not -k (the
    index N / 2 is +N / 2 in both), projected on its own.  A wave with a
    Nyquist component is not transverse at its mirror, so the pin does not
    apply to it; the comparison with the oracle does."""
    from test_oracle_pins import cos_mode
    lib = _lib()
    A, mp = 0.3, 0.8
    lat = lib.Lattice(N, 0.5, 1, "fp64")
    lat.set_background(alpha, "self", mp, 1.0)
    lat.set_potential((0.0, 0.0), (1.0, 0.0), 0.0, 0.0)
    lat.gw_enable(True)
    rng = np.random.default_rng(2)
    f = 1.0 + 0.01 * rng.standard_normal((1, N, N, N))
    lat.set_fields(f, np.zeros_like(f))
    s = np.sin(np.pi * np.array(nvec) / N)
    k = s / np.linalg.norm(s)
    e1 = np.cross(k, [1.0, 0.0, 0.0] if abs(k[0]) < 0.9 else [0.0, 1.0, 0.0])
    e1 /= np.linalg.norm(e1)
    e2 = np.cross(k, e1)
    e = np.outer(e1, e1) - np.outer(e2, e2)
    g = cos_mode(N, 0.5, nvec)
    u = np.stack([A * e[i, j] * g for i, j in G.COMPONENTS])  # a = 1
    lat.gw_set(np.zeros_like(u), u)
    counts, rho, omega, tot = lat.gw_spectrum()
    obs = lat.read_observables()
    lat.close()
    want = mp ** 2 * A ** 2 / 4
    b = int(math.floor(math.sqrt(sum(c * c for c in nvec)) + 0.5))
    if all(abs(c) != N // 2 for c in nvec):
        assert abs(tot - want) <= 1e-12 * want and abs(rho[b] - want) <= 1e-12 * want
    P = L.Params(N=N, dx=0.5, n_fields=1, alpha=alpha, mp=mp)
    rho_tot = sum(obs["EK"][:1]) + sum(obs["EG"][:1]) + obs["EV"]
    oc, orho, oom, otot = G.gw_spectrum(u, 1.0, P, rho_tot=rho_tot, nbins=len(counts))
    assert np.array_equal(counts, oc)
    assert np.max(np.abs(rho - orho)) <= 1e-12 * want
    assert np.max(np.abs(omega - oom)) <= 1e-11 * np.max(np.abs(oom))


def test_gw_axis_wave_sources_no_waves():
    """A scalar plane wave along a lattice axis sources a tensor with no
    transverse-traceless part: the device spectrum stays at round-off while
    the evolved (unprojected) tensor does not."""
    from test_oracle_pins import cos_mode
    lib = _lib()
    N = 16
    lat = lib.Lattice(N, 0.6, 2, "fp64")
    lat.set_potential((0.0, 0.0), (1.0, 0.0), 3.0, 0.0)
    lat.gw_enable(True)
    g = cos_mode(N, 0.6, (2, 0, 0))
    lat.set_fields(np.stack([1.0 + 0.2 * g, 0.1 + 0.1 * g]), np.stack([0.05 * g, 0.02 * g]))
    lat.step("vv4", 0.05, 30)
    v, u = lat.gw_get()
    counts, rho, omega, tot = lat.gw_spectrum()
    lat.close()
    a = 1.0
    unproj = np.mean(np.sum(G.full_tensor(u) ** 2, axis=(0, 1)))
    assert np.max(np.abs(v)) > 1e-4
    assert tot <= 1e-24 * unproj


def test_gw_enable_keeps_state_and_rejects_what_it_cannot_run():
    lib = _lib()
    w = W.C1.with_(N=16, k_ir=2.0, precision="fp64")
    s0 = oracle_seed(w, amp=20.0)
    lat = make_lattice(w)
    lat.set_fields(s0.f, s0.p)
    lat.step("leapfrog", w.dt, 3)
    f0, p0 = lat.get_fields()
    st0 = lat.get_state()
    lat.gw_enable(True)
    f1, p1 = lat.get_fields()
    v, u = lat.gw_get()
    assert np.array_equal(f0, f1) and np.array_equal(p0, p1) and lat.get_state() == st0
    assert not np.any(v) and not np.any(u)
    with pytest.raises(lib.CLError) as e:
        lat.step("rk4", w.dt, 1)
    assert e.value.status == lib.CL_EUNSUPPORTED
    with pytest.raises(lib.CLError) as e:
        lib.Ensemble([lat])
    assert e.value.status == lib.CL_EUNSUPPORTED
    lat.step("leapfrog", w.dt, 2)
    f2, p2 = lat.get_fields()
    lat.gw_enable(False)
    f3, p3 = lat.get_fields()
    assert np.array_equal(f2, f3) and np.array_equal(p2, p3)
    with pytest.raises(lib.CLError) as e:
        lat.gw_get()
    assert e.value.status == lib.CL_ESTATE
    lat.close()


@pytest.mark.parametrize("N,nf,precision", [(8, 1, "fp64"), (16, 2, "fp32"), (32, 1, "fp32"), (64, 2, "fp64")])
def test_observables_leave_the_tensor_out(N, nf, precision):
    """A reduction of a lattice with waves does not load the tensor: it gives the
    observables of the same fields on a lattice without, to the rounding of the
    summation order (FP64 1e-12; FP32 lattices round each thread's plane
    partials, 1e-6)."""
    rng = np.random.default_rng(N)
    f, p = 1.0 + 0.1 * rng.standard_normal((nf, N, N, N)), 0.1 * rng.standard_normal((nf, N, N, N))
    obs = []
    for waves in (False, True):
        lat = _lib().Lattice(N, 0.5, nf, precision)
        if waves:
            lat.gw_enable()
        lat.set_background(expansion="static")
        lat.set_potential(lam=(1.0, 0.5), g2=2.0 if nf == 2 else 0.0)
        lat.set_fields(f, p)
        if waves:
            lat.gw_set(*rng.standard_normal((2, 5, N, N, N)))
        obs.append(lat.read_observables())
        lat.close()
    tol = 1e-12 if precision == "fp64" else 1e-6
    for k in ("EK", "EG", "EV", "mean", "var"):
        a, b = np.asarray(obs[1][k]), np.asarray(obs[0][k])
        assert np.all(np.abs(a - b) <= tol * np.abs(b)), (k, a, b)
