"""Records of a call on their way to the host: calls of up to 256 steps read
them from pinned memory that the closing kernel writes, longer calls copy them
from the device.  Both see the same passes, so the records of the steps that
two calls share are the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nf,integrator", [(3, 2, "vv4"), (3, 1, "leapfrog"), (2, 1, "leapfrog")])
def test_records_of_short_and_long_calls(dim, nf, integrator):
    from paper_2607_24978_amd import _lib as lib
    N = 16
    rng = np.random.default_rng(3)
    f, p = 0.1 * rng.standard_normal((2, nf) + (N,) * dim)
    recs = {}
    for n in (1, 256, 257):
        lat = lib.Lattice(N, 0.5, nf, "fp64", dim=dim)
        lat.set_background(expansion="self")
        lat.set_potential(lam=(1.0, 0.5), g2=2.0 if nf == 2 else 0.0)
        lat.set_fields(f, p)
        recs[n] = lat.step(integrator, 0.01, n)
        state = lat.get_state()
        assert state["step"] == n and state["a"] == recs[n]["a"][-1]
        lat.close()
    for n in (1, 256):
        assert recs[n].shape == (n,) and recs[n].tobytes() == recs[257][:n].tobytes(), n


def test_records_of_many_handles():
    """Handles take their pinned block from shared allocations of eight, some of
    which are kept when their handles are gone: 48 handles, destroyed in another
    order than made and made again from two threads, give the records that each
    of their states has on a handle of its own."""
    import threading
    from paper_2607_24978_amd import _lib as lib
    N, count = 8, 48
    f, p = 0.1 * np.random.default_rng(4).standard_normal((2, count, 1, N, N, N))

    def make(i):
        lat = lib.Lattice(N, 0.5, 1, "fp64")
        lat.set_background(expansion="self")
        lat.set_fields(f[i], p[i])
        return lat

    want = []
    for i in range(count):
        lat = make(i)
        want.append(lat.step("leapfrog", 0.01, 3).tobytes())
        lat.close()

    def check(ids, out):
        lats = {i: make(i) for i in ids}
        for i in reversed(ids):
            out[i] = lats[i].step("leapfrog", 0.01, 3).tobytes()
        for i in ids[::2] + ids[1::2]:
            lats[i].close()

    for split in (1, 2):
        got = {}
        threads = [threading.Thread(target=check, args=(list(range(k, count, split)), got)) for k in range(split)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert [got[i] for i in range(count)] == want
