"""Reads and writes of whole states and sums through the pinned staging slots
(2 MiB each, two per thread, up to sixteen at a time): sizes below, at and past a slot and past
all eight, from one thread and from two."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1010_1233_amd import workloads

pytestmark = pytest.mark.gpu

TAU = workloads.tau_vector(0.8, 1.0, 1.0)
_dp = ctypes.POINTER(ctypes.c_double)
SLOT = 1 << 18  # doubles per slot


def _noalloc(flb, g):
    out = np.full((9, g.ny, g.nx), np.nan)
    assert flb.lib().flb_get_populations_noalloc(g._h, 0, out.ctypes.data_as(_dp),
                                                 out.size) == flb.OK
    return out


# 9 nx ny: two slots less a few values, two and a bit, four and a bit, 28
@pytest.mark.parametrize("nx,ny", [(29126, 2), (233, 250), (257, 455), (901, 899)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_populations_through_the_slots(flb, nx, ny, storage):
    print("slots", nx, ny, storage, flush=True)
    g = flb.Lattice(nx, ny, TAU, 1e-4, u0=(0.03, -0.01), seed=5, storage=storage)
    g.thermalize()
    g.step(3)
    a = g.get_populations()
    assert np.array_equal(a, _noalloc(flb, g))
    h = flb.Lattice(nx, ny, TAU, 1e-4, u0=(0.03, -0.01), seed=6, storage=storage)
    f0 = h.get_populations()[:, :1, :1]
    h.set_populations(a)
    b = h.get_populations()
    if storage == "f32":  # stored values: the round trip is exact
        assert np.array_equal(b, a)
    else:  # the FP32 arithmetic of the codec, then one bfloat16 rounding of f - f0
        assert np.all(np.abs(b - a) <= 2.0 ** -8 * np.abs(a - f0) + 2.0 ** -22)


@pytest.mark.parametrize("model,sides", [("D1Q3", (SLOT // 3 + 1,)), ("D2Q9", (240, 243)),
                                         ("D3Q15", (5, 3, 7)), ("D3Q15", (71, 80, 103))])
def test_other_velocity_sets_through_the_slots(flb, model, sides):
    print("slots", model, sides, flush=True)
    _, _, w, _ = flb.dq_tables(model)
    tau = [1.0] * len(w)
    g = flb.DqLattice(model, sides, tau, 1e-4, seed=3)
    shape = (len(w),) + tuple(reversed(g.sides))
    f = np.random.default_rng(1).normal(0.0, 1e-2, shape) + w.reshape(-1, 1, 1, 1)
    g.set_populations(f)
    # FP32 deviations below 0.08: half a unit in the last place is 2^-28
    assert np.abs(f - w.reshape(-1, 1, 1, 1)).max() < 0.08
    assert np.abs(g.get_populations() - f).max() <= 2.0 ** -28 + 1e-15
    g.step(1)
    a = g.get_populations()
    h = flb.DqLattice(model, sides, tau, 1e-4, seed=3)
    h.set_populations(a)
    assert np.array_equal(h.get_populations(), a)


def test_sums_through_the_slots(flb):
    """The sums of a lattice read whole (several slots) are those of the same
    lattice in a batch, and the normalised ones are the sums times numbers."""
    kw = dict(nx=384, ny=700, tau=TAU, theta=1e-4, u0=(0.02, 0.0), stream_id=2)
    g = flb.Lattice.batch([kw], seed=9)
    b = flb.Lattice.batch([dict(kw, nx=8, ny=9, stream_id=0), kw], seed=9)
    for x in (g, b):
        x.thermalize()
        x.run(20, 10)
    a, n = g.read_correlators()
    assert n == 2 and a.size > 3 * SLOT
    assert np.array_equal(a, b.read_correlators(1)[0])
    r, _ = g.read_normalized_raw()
    V, mu, cs = 384 * 700, 3e-4, 1 / np.sqrt(3.0)
    norm = [1 / (V * mu)] + [1 / (V * 1e-4)] * 6 + [1 / (V * mu * cs)] * 8
    np.testing.assert_allclose(r, a / 2 * np.array(norm)[:, None, None], rtol=1e-14, atol=0)


def test_transfers_from_two_threads(flb):
    """Two handles read and written by two threads at once."""
    g = [flb.Lattice(600 + 50 * i, 500, TAU, 1e-4, seed=i + 1) for i in range(2)]
    want, bad = [], []
    for x in g:
        x.thermalize()
        want.append(x.get_populations())

    def work(i):
        for _ in range(5):
            if not np.array_equal(g[i].get_populations(), want[i]):
                bad.append(i)
            g[i].set_populations(want[i])

    t = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not bad


def test_reads_do_not_wait_for_other_handles(flb):
    """A thread that reads a handle with steps still to run does not hold up
    another handle's read."""
    import time

    import torch
    print("reads beside a busy handle", flush=True)
    busy = flb.Lattice(2048, 2048, TAU, 1e-4, seed=1)
    idle = flb.Lattice(64, 64, TAU, 1e-4, seed=2)
    s = torch.cuda.Stream()
    busy.set_stream(s)
    want = idle.get_populations()
    busy.synchronize()
    end = torch.cuda.Event()
    with torch.cuda.stream(s):
        busy.step(20000)  # about half a second
        end.record()
    t = threading.Thread(target=busy.get_populations)
    t.start()
    time.sleep(0.05)
    got = idle.get_populations()
    early = not end.query()
    t.join()
    assert early and np.array_equal(got, want)
