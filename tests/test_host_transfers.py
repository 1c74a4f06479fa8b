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


CASES = [closing_does_not_wait]


@pytest.mark.parametrize("case", [c.__name__ for c in CASES])
def test_transfers(so, case):
    host_stub.run_case(__file__, case, so)


if __name__ == "__main__":
    host_stub.main({c.__name__: c for c in CASES})
    sys.stdout.flush()
