"""Lattices small enough to step and sample inside one block: the run with
its samples, the same calls one by one, and the general kernels give the same
bits; the sums match the oracle."""
import numpy as np
import pytest

from hip_stream import hip_stream
from paper_1010_1233_amd import workloads

pytestmark = pytest.mark.gpu

TAU = workloads.tau_vector(0.8, 1.1, 0.9)
# the smallest, odd lines, the limits of the rule (sides 64, 1024 sites) and
# just past them (65 x 8, 33 x 32)
SIDES = [(2, 2), (3, 5), (20, 20), (32, 32), (64, 16), (16, 64), (2, 64), (63, 3), (31, 33),
         (65, 8), (33, 32)]


def _make(flb, nx, ny, **kw):
    g = flb.Lattice(nx, ny, TAU, 1e-4, u0=(0.04, -0.01), seed=9, **kw)
    g.thermalize()
    return g


@pytest.mark.parametrize("nx,ny", SIDES)
@pytest.mark.parametrize("storage,ladd", [("f32", False), ("bf16", True), ("f16", False)])
def test_run_equals_single_calls(flb, nx, ny, storage, ladd):
    print("small run", nx, ny, storage, flush=True)
    kw = dict(storage=storage, ladd=ladd, moments=True)
    a, b, c = (_make(flb, nx, ny, **kw) for _ in range(3))
    c.set_time_blocking(1, 64)  # the general step kernels
    a.run(53, 7)
    for i in range(1, 54):
        b.step(1)
        if i % 7 == 0:
            b.accumulate()
    for _ in range(7):
        c.step(7)
        c.accumulate()
    c.step(4)
    for g in (b, c):
        assert np.array_equal(a.get_populations(), g.get_populations())
        assert np.array_equal(a.read_correlators()[0], g.read_correlators()[0])
        assert np.array_equal(a.sample_conservation(), g.sample_conservation())
    a.accumulate()  # a second sample of another state, and one dropped by a reset
    a.step(5)
    b.accumulate()
    b.step(5)
    assert np.array_equal(a.read_correlators()[0], b.read_correlators()[0])
    a.accumulate()
    a.reset_correlators()
    a.step(4)
    assert a.read_correlators()[1] == 0 and not a.read_correlators()[0].any()


@pytest.mark.parametrize("nx,ny", SIDES)
def test_sums_match_the_oracle(flb, oracle_lib, nx, ny):
    print("small oracle", nx, ny, flush=True)
    g = _make(flb, nx, ny, moments=True)
    o = oracle_lib.Lattice(nx, ny, TAU, 1e-4, u0=(0.04, -0.01), seed=9, moments=True)
    o.thermalize()
    g.run(30, 3)
    for _ in range(10):
        o.step(3)
        o.sample()
    acc, n = g.read_correlators()
    assert n == 10 and np.all(acc[:, 0, 0] == 0)
    want = np.concatenate([o.acc, o.acc_m])
    scale = np.abs(want).reshape(21, -1).max(axis=1)
    for q in range(21):
        assert np.abs(acc[q] - want[q]).max() <= 2e-4 * max(scale[q], scale[:5].max() * 1e-3), q


def test_batch_of_small_and_large_equals_alone(flb):
    """Small lattices stepped resident (a batch of them), in a batch with a
    large one (general step kernels) and alone: the same bits."""
    specs = [dict(nx=nx, ny=ny, tau=TAU, theta=1e-4, u0=(0.01 * i, 0.0), stream_id=i)
             for i, (nx, ny) in enumerate(SIDES[:9])]
    big = dict(nx=100, ny=70, tau=TAU, theta=1e-4, stream_id=50)
    for storage in ("f32", "bf16"):
        a = flb.Lattice.batch(specs, seed=4, storage=storage)
        b = flb.Lattice.batch(specs[:4] + [big] + specs[4:], seed=4, storage=storage)
        for g in (a, b):
            g.thermalize()
            g.run(47, 5)
        for i in range(9):
            j = i + (i >= 4)
            assert np.array_equal(a.get_populations(i), b.get_populations(j)), i
            assert np.array_equal(a.read_correlators(i)[0], b.read_correlators(j)[0]), i
            assert np.array_equal(a.sample_conservation(i), b.sample_conservation(j)), i
        one = flb.Lattice.batch([specs[2]], seed=4, storage=storage)
        one.thermalize()
        one.run(47, 5)
        assert np.array_equal(one.read_correlators()[0], a.read_correlators(2)[0])


def test_more_lattices_than_compute_units(flb):
    """600 lattices (the sums stay in memory or in LDS by the block's size)
    and one alone: the same bits; a launch's step limit is crossed."""
    specs = [dict(nx=20, ny=20, tau=TAU, theta=1e-4, stream_id=i) for i in range(600)]
    a = flb.Lattice.batch(specs, seed=4, moments=True)
    b = flb.Lattice.batch(specs[599:], seed=4, moments=True)
    for g in (a, b):
        g.thermalize()
        g.run(8200, 41)
    assert np.array_equal(a.get_populations(599), b.get_populations(0))
    assert np.array_equal(a.read_correlators(599)[0], b.read_correlators(0)[0])


@pytest.mark.parametrize("nx,ny", [(20, 20), (33, 32)])
@pytest.mark.parametrize("n", [4, 6])
def test_samples_follow_the_callers_time_after_replays(flb, nx, ny, n):
    """Replays of captured steps advance the noise counter, not the handle's
    time: a run's samples are those of its own time, in count and in place."""
    import torch
    print("samples after replays", nx, ny, n, flush=True)
    got = []
    for one_step in (False, True):
        g = _make(flb, nx, ny)
        if one_step:
            g.set_time_blocking(1, 64)  # the general step kernels
        with hip_stream(flb) as s:
            g.set_stream(s)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s):
                g.step(n)
            with torch.cuda.stream(s):
                for _ in range(3):
                    graph.replay()
            g.set_stream(None)
        assert g.t == n
        counts = []
        for steps, every in ((2, 10), (8, 10), (7, 7), (23, 5)):
            g.run(steps, every)
            counts.append(g.read_correlators()[1])
        assert counts == [(n + 2) // 10, 1, 1 + (n + 17) // 7 - (n + 10) // 7,
                          1 + (n + 17) // 7 - (n + 10) // 7 + (n + 40) // 5 - (n + 17) // 5]
        got.append((g.get_populations(), *g.read_correlators(), g.sample_conservation()))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
