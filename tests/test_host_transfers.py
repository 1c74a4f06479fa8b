"""Transfers between handles and host memory, their host side alone: who waits
for whom, and which pinned memory is held when (no GPU: see host_stub)."""
import sys
import threading

import pytest

import host_stub

TAU = [1.0] * 9


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_stub.build(tmp_path_factory.mktemp("stub"))


def _start(fn):
    t = threading.Thread(target=fn, daemon=True)
    t.start()
    return t


def closing_does_not_wait(s):
    """A read that waits for its stream's steps does not hold up the closing of
    another handle."""
    a, b = (s.flb.Lattice(20, 20, TAU, 1e-4) for _ in range(2))
    stream = s.stream()
    a.set_stream(stream)
    s.hold("hipStreamSynchronize", stream)
    reader = _start(a.get_populations)
    assert s.held("hipStreamSynchronize")
    closer = _start(b.close)
    closer.join(5)
    assert not closer.is_alive() and reader.is_alive()
    s.release("hipStreamSynchronize")
    reader.join(5)
    assert not reader.is_alive()


def last_close_beside_a_new_handle(s):
    """A handle opened and read while the last one before it closes keeps its
    slots (freed ones fault when touched)."""
    def values(g):
        return g.get_populations()

    def read_new():
        b = s.flb.Lattice(400, 400, TAU, 1e-4)  # several chunks
        values(b)
        done.append(b)

    done = []
    a = s.flb.Lattice(400, 400, TAU, 1e-4)
    values(a)
    s.hold("hipHostFree")
    closer = _start(a.close)
    assert s.held("hipHostFree")
    s.hold("hipEventSynchronize")
    reader = _start(read_new)
    assert s.held("hipEventSynchronize")  # its first chunks are under way
    s.release("hipHostFree")
    closer.join(5)
    assert not closer.is_alive()
    s.release("hipEventSynchronize")
    reader.join(5)
    assert done
    done.pop().close()
    assert s.L.hs_pinned_now() == 0


def many_handles_come_and_go(s):
    """Threads that open, read and close handles of their own, some of several
    chunks: nothing is left behind."""
    bad = []

    def work(i):
        try:
            for k in range(30):
                side = 300 if (i + k) % 3 == 0 else 20
                g = s.flb.Lattice(side, side, TAU, 1e-4)
                g.get_populations()
                g.close()
        except BaseException as e:  # noqa: B902
            bad.append(e)

    threads = [_start(lambda i=i: work(i)) for i in range(6)]
    for t in threads:
        t.join(60)
        assert not t.is_alive()
    assert not bad
    assert s.L.hs_pinned_now() == 0


def more_transfers_than_slot_pairs(s):
    """Eleven reads at once of handles with steps to run: the main slots, seven
    pairs more, and three that wait for the main slots; all end."""
    gs = [s.flb.Lattice(20, 20, TAU, 1e-4) for _ in range(11)]
    s.hold("hipStreamSynchronize")
    readers = [_start(g.get_populations) for g in gs]
    assert s.held("hipStreamSynchronize", 8)
    assert not s.held("hipStreamSynchronize", 9, 300)
    s.release("hipStreamSynchronize")
    for t in readers:
        t.join(10)
        assert not t.is_alive()
    for g in gs:
        g.close()
    assert s.L.hs_pinned_now() == 0


def slots_are_made_as_needed(s):
    """A small read pins little, a large one what it uses (4 MiB a thread), and
    all of it is kept until the last handle closes."""
    MiB = 1 << 20
    a = s.flb.Lattice(20, 20, TAU, 1e-4)
    assert s.L.hs_pinned_now() == 0
    a.get_populations()
    small = s.L.hs_pinned_now()
    assert 9 * 400 * 8 < small <= MiB
    a.set_populations(a.get_populations())
    a.read_correlators()
    assert s.L.hs_pinned_now() == small
    for side, pairs in ((100, 1), (200, 1), (256, 2), (2048, 8), (300, 8)):
        b = s.flb.Lattice(side, side, TAU, 1e-4)
        b.get_populations()
        assert s.L.hs_pinned_now() == small + pairs * 4 * MiB, side
        b.close()
    assert not any(x.startswith("hipHostFree") for x in s.take_log())
    a.close()
    assert s.L.hs_pinned_now() == 0


def current_device_of_the_caller(s):
    """A handle of one device read and written while another is the caller's
    current one, which stays so."""
    import ctypes
    s.L.hipSetDevice(1)
    gs = [s.flb.Lattice(side, side, TAU, 1e-4) for side in (20, 250, 700)]
    gs.append(s.flb.DqLattice("D1Q3", (1 << 12,), [1.0] * 3, 1e-4))
    s.L.hipSetDevice(0)
    for g in gs:
        g.set_populations(g.get_populations())
        g.read_correlators()
        d = ctypes.c_int(-1)
        s.L.hipGetDevice(ctypes.byref(d))
        assert d.value == 0


CASES = [current_device_of_the_caller, slots_are_made_as_needed, closing_does_not_wait, last_close_beside_a_new_handle, many_handles_come_and_go,
         more_transfers_than_slot_pairs]


@pytest.mark.parametrize("case", [c.__name__ for c in CASES])
def test_transfers(so, case):
    host_stub.run_case(__file__, case, so)


if __name__ == "__main__":
    host_stub.main({c.__name__: c for c in CASES})
    sys.stdout.flush()
