"""Samples beside the steps that follow them, on lattices of at least 2^21
sites, where they run on a second stream: with the library's own grouping of
the steps (marching launches of four and five steps) and with one, two and
three steps per launch, the same bits as with samples enqueued at once
(sample overlap off)."""
import numpy as np
import pytest

from paper_1010_1233_amd import workloads

pytestmark = pytest.mark.gpu

TAU = workloads.tau_vector(0.7, 0.9, 1.0)
# one lattice; one with lattices of a single block and of Bluestein lines beside it
BATCHES = {"one": [(2048, 1100)], "mixed": [(20, 20), (2048, 1024), (300, 200), (7, 64)]}
STEPS = (1, 5, 4, 10, 3, 16, 2)


def _pair(flb, sides, storage, moments, blocking):
    specs = [dict(nx=nx, ny=ny, tau=TAU, theta=1e-4, u0=(0.03, -0.01), stream_id=i)
             for i, (nx, ny) in enumerate(sides)]
    hs = [flb.Lattice.batch(specs, seed=21, storage=storage, moments=moments) for _ in range(2)]
    hs[1].set_sample_overlap(False)
    for g in hs:
        if blocking:
            g.set_time_blocking(blocking, 64)
        g.thermalize()
    return hs


@pytest.mark.parametrize("blocking", [0, 1, 2, 3])
@pytest.mark.parametrize("storage,moments", [("f32", False), ("f32", True), ("bf16", False),
                                             ("bf16", True)])
@pytest.mark.parametrize("batch", sorted(BATCHES))
def test_samples_beside_large_steps_equal_immediate(flb, batch, storage, moments, blocking):
    print("large overlap", batch, storage, moments, blocking, flush=True)
    a, b = _pair(flb, BATCHES[batch], storage, moments, blocking)
    for n in STEPS:  # the overwriting launch absent, or the second of two to sixteen
        for g in (a, b):
            g.step(n)
            g.accumulate()
    for g in (a, b):
        g.run(47, 10)
        g.run(9, 2)
    for i in range(len(BATCHES[batch])):
        (ra, na), (rb, nb) = a.read_correlators(i), b.read_correlators(i)
        assert na == nb and np.array_equal(ra, rb), i
        assert np.array_equal(a.get_populations(i), b.get_populations(i)), i
        assert np.array_equal(a.sample_conservation(i), b.sample_conservation(i)), i
