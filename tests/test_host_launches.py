"""Which launches the library's host side makes of a caller's calls (no GPU:
see host_stub)."""
import pytest

import host_stub

TAU = [1.0] * 9
# one block's lattice, small tiles, tiles of three and two steps, marching waves
SIDES = [(20, 20), (256, 256), (700, 500), (2048, 2048)]
CALLS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 20, 25, 37, 100)


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_stub.build(tmp_path_factory.mktemp("stub"))


def _flips(s, call):
    """Buffer flips of a call's step launches, each reading what the one
    before it wrote."""
    s.take_log()
    call()
    steps = s.take_steps()
    for a, b in zip(steps, steps[1:]):
        assert a[3] == b[2] and a[2] == b[3]
    return len(steps)


def captured_steps_keep_the_buffers(s):
    """Each call while a stream is captured, and each one after it (between
    replays), leaves the state in the buffer that one-step launches would."""
    for storage in ("f32", "bf16"):
        for nx, ny in SIDES:
            g = s.flb.Lattice(nx, ny, TAU, 1e-4, storage=storage)
            stream = s.stream()
            g.set_stream(stream)
            g.reset_correlators()  # set up, which a capture does not allow
            for capturing in (1, 0):
                s.L.hs_capture(stream, capturing)
                for n in CALLS:
                    assert _flips(s, lambda: g.step(n)) % 2 == n % 2, (nx, storage, capturing, n)
                    g.accumulate()
                    assert _flips(s, lambda: g.step(n)) % 2 == n % 2, (nx, storage, capturing, n)
                    for every in (1, 3, 4, 10):
                        flips = _flips(s, lambda: g.run(n, every))
                        assert flips % 2 == n % 2, (nx, storage, capturing, n, every)
            g.close()


def handles_never_captured_are_grouped_freely(s):
    """Launches of steps from one buffer into the other (resident steps make
    none)."""
    for sides, n, launches in ((SIDES[0], 8, 0), (SIDES[0], 3, 1), (SIDES[1], 4, 1),
                               (SIDES[2], 6, 2), (SIDES[3], 4, 1), (SIDES[3], 15, 3)):
        g = s.flb.Lattice(*sides, TAU, 1e-4)
        assert _flips(s, lambda: g.step(n)) == launches, (sides, n)
        g.close()


def captured_line_steps_keep_the_buffers(s):
    """The same for the lines that take several steps a launch."""
    g = s.flb.DqLattice("D1Q3", (3000,), [1.0] * 3, 0.0)
    stream = s.stream()
    g.set_stream(stream)
    assert _flips(s, lambda: g.step(16)) == 2
    for capturing in (1, 0):
        s.L.hs_capture(stream, capturing)
        for n in CALLS:
            s.take_log()
            g.step(n)
            steps = s.take_steps()
            assert len(steps) % 2 == n % 2 and len(steps) <= n, (capturing, n)
            assert sum(x[1] for x in steps) == n and all(1 <= x[1] <= 8 for x in steps)


def timed_launches(s):
    """Launch timing counts the launches of a run outside its whole periods, and
    no sample's."""
    s.cost("small_kernel<0, true, false>", 1.0)
    s.cost("patch_kernel", 1.0)
    s.cost("corr_rows", 100.0)
    for sides in SIDES[:2]:
        g = s.flb.Lattice(*sides, TAU, 1e-4)
        g.set_launch_timing(True)
        for steps, every, launches in ((7, 10, 1), (3, 10, 1), (30, 10, 0), (2, 10, 1),
                                       (8, 10, 1), (25, 10, 1), (14, 20, 2)):
            t = g.t
            g.run(steps, every)
            n, ms = g.launch_timing()
            assert n == launches and ms == launches, (sides, steps, every, t, n, ms)
            assert g.t == t + steps
        g.accumulate()
        s.take_log()
        g.step(8)
        small = [x for x in s.take_log() if "launch small_kernel" in x]
        n, ms = g.launch_timing()
        assert (n, ms) == (1, 1.0) and len(small) == (2 if sides == SIDES[0] else 0)
        g.set_launch_timing(False)
        g.run(100, 10)
        assert g.launch_timing() == (0, 0.0)


def a_tuned_grouping_runs_what_was_timed(s):
    """The tuner keeps the library's own grouping: its launches stay those that
    it timed, while the handle reports the fastest shape that can be set, which
    is what it runs once a caller names one."""
    s.cost("march_kernel", 0.01)
    s.cost("patch_kernel", 0.01)
    s.cost("step3_kernel<0, true, true, 128", 0.5)
    s.cost("step", 1.0)
    for sides in SIDES[1:2] + SIDES[3:]:
        plain, tuned, other = (s.flb.Lattice(*sides, TAU, 1e-4) for _ in range(3))
        other.autotune(12)
        for tune in (lambda: tuned.autotune(12), lambda: tuned.autotune_path(12, 10)):
            tune()
            s.take_log()
            got = []
            for g in (plain, tuned):
                names = []
                for n in (1, 2, 3, 6, 10, 11):
                    s.take_log()
                    g.step(n)
                    names += [x.split(" stream=")[0] for x in s.take_log()]
                got.append(names)
            assert got[0] == got[1]
            assert tuned.time_blocking() == (3, 128) and tuned.step_config()[2]
            assert list(tuned.lattice_tiles()) == [128]
        shape = tuned.step_config()
        tuned.set_time_blocking(2, 32)
        assert tuned.step_config() == shape and tuned.time_blocking() == (2, 32)
        shape = other.step_config()
        other.set_step_config(*shape)
        assert other.step_config() == shape and other.time_blocking() == (3, 128)
        s.take_log()
        other.step(3)
        assert [x[0] for x in s.take_steps()] == ["step3_kernel"]


def samples_beside_the_steps(s):
    """From 2^21 sites on a sample runs on a second stream: behind the work
    before it, read before the second step launch writes its state, and done
    before the step call's work is.  Smaller lattices' samples come before the
    steps, on their stream."""
    def events(lines, kind, stream):
        return [(i, x.split("event=")[1]) for i, x in enumerate(lines)
                if x.startswith(f"{kind} stream={stream:#x}")]

    def launches(lines, part, stream):
        return [i for i, x in enumerate(lines)
                if x.startswith("launch " + part) and f"stream={stream:#x} " in x]

    for sides, blocking in ((SIDES[3], 0), (SIDES[3], 1), (SIDES[3], 2), (SIDES[3], 3),
                            (SIDES[2], 0)):
        g = s.flb.Lattice(*sides, TAU, 1e-4, moments=True)
        if blocking:
            g.set_time_blocking(blocking, 64)
        main = s.stream()
        g.set_stream(main)
        for n in (1, 5, 10, 16):
            g.accumulate()
            s.take_log()
            g.step(n)
            lines = s.take_log()
            steps = [i for p in ("step", "march") for i in launches(lines, p, main)]
            steps.sort()
            other = {int(x.split("stream=")[1].split()[0], 16) for x in lines if "stream=" in x}
            other.discard(main)
            if sides != SIDES[3]:
                assert not other
                assert max(launches(lines, "corr_", main)) < min(steps)
                continue
            (aux,) = other
            rows = launches(lines, "corr_", aux)
            assert rows and not launches(lines, "corr_", main)
            (fork, e0), (back, e0b) = events(lines, "record", main)[0], events(lines, "wait", aux)[0]
            assert e0 == e0b and fork < back < min(rows)
            (read, e1), (done, e2) = events(lines, "record", aux)
            # every kernel that reads the state comes before the first record
            readers = [i for i in rows if "moment_fields" in lines[i] or "corr_rows" in lines[i]]
            assert readers and max(readers) < read and max(rows) < done
            waits = events(lines, "wait", main)
            assert waits[-1][1] == e2 and waits[-1][0] > max(steps)
            assert len(waits) == (2 if len(steps) > 1 else 1)
            if len(steps) > 1:
                assert waits[0][1] == e1 and steps[0] < waits[0][0] < steps[1]
                assert read < waits[0][0]
        g.close()


CASES = [samples_beside_the_steps, a_tuned_grouping_runs_what_was_timed, timed_launches, captured_steps_keep_the_buffers, captured_line_steps_keep_the_buffers,
         handles_never_captured_are_grouped_freely]


@pytest.mark.parametrize("case", [c.__name__ for c in CASES])
def test_launches(so, case):
    host_stub.run_case(__file__, case, so)


if __name__ == "__main__":
    host_stub.main({c.__name__: c for c in CASES})
