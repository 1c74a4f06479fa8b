"""GPU parity of the fused step against the FP64 oracle (through the C ABI).

Bars: the Philox words are bit-exact; the normals agree to |dz| <= 2e-5 (FP32
hardware log/sqrt/sin/cos vs FP64 libm); populations agree to 1e-6 rho0 after
one step and to 1e-5 rho0 after 10^3 steps (FP32 storage); the launch shape
never changes a result (bit-identical across tiles, batches and graphs).
"""
import sys

import numpy as np
import pytest

from hip_stream import hip_stream
from paper_1010_1233_amd import workloads

pytestmark = pytest.mark.gpu

TAU_C1 = workloads.tau_vector(0.8, 0.8, 1.0)


def note(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def pair(flb, oracle_lib, nx, ny, tau, theta, u0=(0.0, 0.0), seed=1, stream_id=0, ladd=False,
         storage="f32", rho0=1.0):
    g = flb.Lattice(nx, ny, tau, theta, rho0=rho0, u0=u0, seed=seed, storage=storage,
                    stream_id=stream_id, ladd=ladd)
    o = oracle_lib.Lattice(nx, ny, tau, theta, rho0=rho0, u0=u0, seed=seed, stream_id=stream_id,
                           ladd=ladd)
    return g, o


@pytest.mark.parametrize("seed,stream_id,t", [(1, 0, 0), (0xDEADBEEFCAFEF00D, 7, 123456),
                                              (5, 95, 0xFFFFFFFE)])
def test_noise_words_bit_exact_and_normals_close(flb, oracle_lib, seed, stream_id, t):
    note("noise", seed, stream_id, t)
    g = flb.Lattice(64, 64, TAU_C1, 1e-4, seed=seed, stream_id=stream_id)
    n = 1 << 16
    site0 = 1000
    w, z = g.debug_noise(t, site0, n)
    idx = np.r_[0:2000, n - 2000:n]
    for k in idx:
        ow = oracle_lib.noise_words(seed, stream_id, t, site0 + int(k), 0)
        assert w[k].tolist() == ow.tolist(), k
    zo = np.array([oracle_lib.normals_from_words(w[k]) for k in range(n)])
    err = np.abs(z.astype(np.float64) - zo)
    note("max |dz|", err.max())
    assert err.max() <= 5e-6  # measured 6.6e-7 on MI355X
    g.close()


def test_initial_state_is_the_equilibrium(flb, oracle_lib):
    g, o = pair(flb, oracle_lib, 17, 9, TAU_C1, 1e-4, u0=(0.05, -0.02))
    f = g.get_populations()
    assert np.abs(f - o.f).max() < 1e-7


@pytest.mark.parametrize("nx,ny", [(37, 23), (2, 2), (3, 5), (257, 3), (64, 64), (1000, 7),
                                   (5, 300)])
def test_one_step_from_random_state(flb, oracle_lib, nx, ny):
    note("one step", nx, ny)
    tau = workloads.tau_vector(0.7, 1.1, 1.3)
    g, o = pair(flb, oracle_lib, nx, ny, tau, 1e-3, u0=(0.03, 0.01), seed=9, stream_id=3)
    f0 = workloads.perturbed(oracle_lib.equilibrium(1.0, 0.03, 0.01), nx, ny, 0.01, seed=nx * ny)
    g.set_populations(f0)
    o.set_populations(f0)
    assert np.abs(g.get_populations() - f0).max() < 1e-7
    for _ in range(3):
        g.step(1)
        o.step(1)
        err = np.abs(g.get_populations() - o.f).max()
        note("  max |df|", err)
        assert err < 1e-6


def test_thousand_steps_config1(flb, oracle_lib):
    """32^2, rho0 = 1, tau (.8,.8,1), theta = 1e-4, seed 1: max|df| <= 1e-5 rho0
    after 10^3 steps."""
    c = workloads.CONFIGS["c1_32"]
    g, o = pair(flb, oracle_lib, c["nx"], c["ny"], c["tau"], c["theta"], seed=c["seed"])
    g.step(1000)
    o.step(1000)
    err = np.abs(g.get_populations() - o.f).max()
    note("c1 1e3 steps max |df|", err)
    assert err <= 1e-5 * c["rho0"]
    assert g.t == 1000


def test_thousand_steps_mean_flow_and_thermal_start(flb, oracle_lib):
    tau = workloads.tau_vector(0.6, 1.0, 1.0)
    g, o = pair(flb, oracle_lib, 48, 40, tau, 1e-4, u0=(0.05, 0.0), seed=5, stream_id=2)
    g.thermalize()
    o.thermalize()
    assert np.abs(g.get_populations() - o.f).max() < 1e-7
    g.step(1000)
    o.step(1000)
    err = np.abs(g.get_populations() - o.f).max()
    note("mean flow 1e3 steps max |df|", err)
    assert err <= 1e-5


def test_ghost_noise_switch(flb, oracle_lib):
    g, o = pair(flb, oracle_lib, 20, 20, workloads.tau_vector(1, 1, 1), 1e-4, ladd=True)
    g.step(200)
    o.step(200)
    assert np.abs(g.get_populations() - o.f).max() <= 1e-5


def test_noise_free_uniform_state_stays(flb):
    g = flb.Lattice(64, 32, workloads.tau_vector(0.6, 0.9, 1.3), 0.0, u0=(0.1, 0.03))
    f0 = g.get_populations()
    g.step(500)
    assert np.abs(g.get_populations() - f0).max() <= 1e-6


def test_conservation_sums_match_oracle(flb, oracle_lib):
    g, o = pair(flb, oracle_lib, 40, 30, TAU_C1, 1e-3, u0=(0.02, 0.0), seed=3)
    g.thermalize()
    o.thermalize()
    c0 = g.conservation()
    assert np.abs(c0 - o.conservation()).max() < 1e-5
    g.step(1001)
    o.step(1001)
    cg, co = g.conservation(), o.conservation()
    note("conservation gpu", cg, "oracle", co)
    assert np.abs(cg - co).max() < 2e-5
    # mass and momentum stay put (FP32 storage: rounding random walk only)
    assert np.abs(cg[:3] - c0[:3]).max() < 1e-3
    # staggered momenta flip sign every step (even sides)
    assert np.allclose(cg[3:], -c0[3:], atol=1e-4)


def test_conservation_flags_nan(flb, oracle_lib):
    g = flb.Lattice(8, 8, TAU_C1, 1e-4)
    f = g.get_populations()
    f[4, 3, 5] = np.nan
    g.set_populations(f)
    assert not np.all(np.isfinite(g.conservation()))


@pytest.mark.parametrize("cfg", [(64, 1, 0), (128, 1, 1), (256, 1, 0), (64, 2, 1), (128, 2, 0),
                                 (256, 2, 1), (64, 4, 0), (128, 4, 1), (256, 4, 0)])
def test_launch_shape_does_not_change_results(flb, cfg):
    """Every (threads along x, sites per thread, streaming stores) shape gives
    bit-identical states in every storage format; 301 and 1000 columns leave
    ragged groups at row ends."""
    for storage in ("f32", "f16", "bf16"):
        for nx, ny in ((301, 37), (1000, 7)):
            ref = flb.Lattice(nx, ny, TAU_C1, 1e-3, u0=(0.03, -0.02), seed=4, storage=storage)
            ref.set_step_config(256, 1, 0)
            ref.thermalize()
            ref.step(20)
            a = ref.get_populations()
            g = flb.Lattice(nx, ny, TAU_C1, 1e-3, u0=(0.03, -0.02), seed=4, storage=storage)
            g.set_step_config(*cfg)
            assert g.step_config() == (cfg[0], cfg[1], bool(cfg[2]))
            g.thermalize()
            g.step(20)
            assert np.array_equal(g.get_populations(), a), (storage, nx, ny)


def test_batch_equals_separate_lattices(flb):
    specs = [dict(nx=33, ny=20, tau=TAU_C1, theta=1e-3, u0=(0.0, 0.0), stream_id=0),
             dict(nx=64, ny=64, tau=workloads.tau_vector(0.6, 1.0, 1.0), theta=1e-4,
                  u0=(0.05, 0.0), stream_id=1),
             dict(nx=7, ny=129, tau=workloads.tau_vector(1.2, 0.9, 0.7), theta=2e-4,
                  u0=(0.0, -0.03), stream_id=2)]
    b = flb.Lattice.batch(specs, seed=11)
    assert b.nlattices == 3
    b.thermalize()
    b.step(57)
    for i, s in enumerate(specs):
        g = flb.Lattice(s["nx"], s["ny"], s["tau"], s["theta"], u0=s["u0"], seed=11,
                        stream_id=s["stream_id"])
        g.thermalize()
        g.step(57)
        assert np.array_equal(b.get_populations(i), g.get_populations()), i


def test_torch_stream_binding(flb):
    torch = pytest.importorskip("torch")
    s = torch.cuda.Stream()
    a = flb.Lattice(40, 40, TAU_C1, 1e-3, seed=2)
    a.set_stream(s)
    a.step(30)
    a.synchronize()
    b = flb.Lattice(40, 40, TAU_C1, 1e-3, seed=2)
    b.step(30)
    assert np.array_equal(a.get_populations(), b.get_populations())


def test_large_lattice_one_step(flb, oracle_lib):
    """4096^2 (the 16.8M-site workload, u0_x = 0.05, tau_s = 0.6) in the
    default one-step launch shape: one full step against the oracle at every
    site.  The two-step shape the benchmark times is checked against the
    oracle at sampled sites in test_sampled_sites_at_full_and_maximum_size."""
    c = workloads.CONFIGS["c5_4096"]
    note("4096^2 one step")
    g, o = pair(flb, oracle_lib, c["nx"], c["ny"], c["tau"], c["theta"], u0=c["u0"],
                seed=c["seed"])
    f0 = workloads.perturbed(oracle_lib.equilibrium(1.0, *c["u0"]), c["nx"], c["ny"], 3e-3,
                             seed=12)
    g.set_populations(f0)
    o.set_populations(f0)
    del f0
    g.step(1)
    o.step(1)
    err = np.abs(g.get_populations() - o.f).max()
    note("4096^2 max |df|", err)
    assert err < 1e-6


def test_16bit_storage_tracks_oracle(flb, oracle_lib):
    """BF16 / FP16 scaled deviations: quantisation error of the stored state
    only (relative to the fluctuation scale sqrt(mu rho0 w_i))."""
    tau = workloads.tau_vector(0.8, 1.0, 1.0)
    for storage, tol in (("f16", 2e-3), ("bf16", 2e-2)):
        g, o = pair(flb, oracle_lib, 32, 32, tau, 1e-4, storage=storage, seed=6)
        assert g.storage_info() == (flb.STORAGE[storage], 2)
        g.thermalize()
        o.thermalize()
        g.step(100)
        o.step(100)
        sc = np.sqrt(3e-4 * 4 / 9)
        err = np.abs(g.get_populations() - o.f).max() / sc
        note(storage, "relative err", err)
        assert err < tol * 100 ** 0.5


def test_invalid_calls_report_errors(flb):
    g = flb.Lattice(8, 8, TAU_C1, 1e-4)
    with pytest.raises(flb.FlbError):
        g.step(-1)
    with pytest.raises(flb.FlbError):
        g.conservation(lattice=3)
    with pytest.raises(flb.FlbError):
        g.set_step_config(100, 1, 0)
    import ctypes
    buf = np.zeros(10)
    rc = flb.lib().flb_read_correlators(g._h, 0, buf.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                                        10, None)
    assert rc == flb.ESIZE


def test_autotune_keeps_state_and_caches(flb, tmp_path, monkeypatch):
    monkeypatch.setenv("FLB_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    ref = flb.Lattice(257, 130, TAU_C1, 1e-3, seed=12)
    g = flb.Lattice(257, 130, TAU_C1, 1e-3, seed=12)
    for h in (ref, g):
        h.thermalize()
        h.step(5)
    cfg, ms = g.autotune(3)
    assert ms > 0 and cfg[0] in (64, 128, 256) and cfg[1] in (1, 2, 4)
    assert g.t == 5
    assert np.array_equal(g.get_populations(), ref.get_populations())
    g.step(7)
    ref.step(7)
    assert np.array_equal(g.get_populations(), ref.get_populations())
    lines = (tmp_path / "tune.txt").read_text().splitlines()
    assert len(lines) == 1
    # second handle of the same shape: the choice comes from the cache file
    h = flb.Lattice(257, 130, TAU_C1, 1e-3, seed=1)
    cfg2, ms2 = h.autotune(3)
    assert cfg2 == cfg and abs(ms2 - ms) < 1e-5  # cached with 6 decimals
    assert h.time_blocking() == g.time_blocking()
    assert len((tmp_path / "tune.txt").read_text().splitlines()) == 1


def test_autotune_path_keeps_state_and_sums(flb, tmp_path, monkeypatch):
    """Tuning on whole sampling periods: the populations, the step counter
    and the correlator sums are as before (the run after it has the bits of
    an untuned handle set to the chosen shape); refused once a sample has
    been taken; cached under its own key."""
    monkeypatch.setenv("FLB_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    kw = dict(u0=(0.02, 0.0), seed=21)
    ref = flb.Lattice(300, 128, TAU_C1, 1e-3, **kw)
    g = flb.Lattice(300, 128, TAU_C1, 1e-3, **kw)
    for h in (ref, g):
        h.thermalize()
        h.step(4)
    cfg, ms = g.autotune_path(4, 5)
    assert ms > 0 and cfg[0] in (64, 128, 256) and cfg[1] in (1, 2, 4)
    assert g.t == 4
    assert np.array_equal(g.get_populations(), ref.get_populations())
    with pytest.raises(flb.FlbError):
        g.sample_conservation()  # the tuning's samples were dropped
    ref.set_step_config(*cfg)
    ref.set_time_blocking(*g.time_blocking())
    for h in (ref, g):
        h.run(20, 5)
    a, na = g.read_correlators()
    b, nb = ref.read_correlators()
    assert na == nb == 4 and np.array_equal(a, b)
    assert np.array_equal(g.get_populations(), ref.get_populations())
    with pytest.raises(flb.FlbError):
        g.autotune_path(4, 5)  # samples taken
    g.reset_correlators()
    cfg2, ms2 = g.autotune_path(4, 5)  # from the cache file
    assert cfg2 == cfg and abs(ms2 - ms) < 1e-5
    lines = (tmp_path / "tune.txt").read_text().splitlines()
    assert len(lines) == 1 and lines[0].startswith("flb-path:")


def test_autotune_cache_with_lattice_tiles(flb, tmp_path, monkeypatch):
    """A cache line naming per-lattice tiles ("L" and each lattice's log2
    width) is taken as it stands: the handle steps with those tiles and
    gives the bits of an untuned handle set to them; a line whose lattice
    count does not match, or whose widths are not 32 or 64, is skipped."""
    sides = [(70, 40), (33, 129), (8, 8)]
    specs = [dict(nx=nx, ny=ny, tau=TAU_C1, theta=1e-3, stream_id=i)
             for i, (nx, ny) in enumerate(sides)]
    total = sum(nx * ny for nx, ny in sides)
    key = f"flb-path:0:{len(sides)}:{total}:{max(max(x) for x in sides)}:1:5"
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{key} 128 1 1 2 L565 0.5\n"
                     f"{key} 128 1 1 2 L56 0.25\n"     # wrong lattice count
                     f"{key} 128 1 1 2 L575 0.125\n")  # width 2^7 not offered
    monkeypatch.setenv("FLB_AUTOTUNE_CACHE", str(cache))
    g = flb.Lattice.batch(specs, seed=8)
    cfg, ms = g.autotune_path(4, 5)
    assert cfg == (128, 1, True) and ms == 0.5
    assert g.time_blocking() == (2, 0) and g.lattice_tiles() == [32, 64, 32]
    ref = flb.Lattice.batch(specs, seed=8)
    ref.set_step_config(128, 1, 1)
    ref.set_lattice_tiles([32, 64, 32])
    for h in (g, ref):
        h.thermalize()
        h.run(23, 5)
    for i in range(len(sides)):
        assert np.array_equal(g.get_populations(i), ref.get_populations(i))


def test_resume_from_saved_state_is_bit_identical(flb):
    """Checkpoint = populations + t (the noise is counter-based): a new handle
    given both continues exactly like the uninterrupted run."""
    ref = flb.Lattice(40, 24, TAU_C1, 1e-3, u0=(0.02, 0.0), seed=77, stream_id=5)
    ref.thermalize()
    ref.step(123)
    saved, t = ref.get_populations(), ref.t
    ref.step(50)
    g = flb.Lattice(40, 24, TAU_C1, 1e-3, u0=(0.02, 0.0), seed=77, stream_id=5)
    g.set_populations(saved)
    g.t = t
    assert g.t == 123
    g.step(50)
    assert np.array_equal(g.get_populations(), ref.get_populations())
    with pytest.raises(flb.FlbError):
        g.t = -1


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_time_blocking_equals_one_step_launches(flb, storage):
    """Two and three steps per launch (halo recomputed on chip) give exactly
    the populations of one step per launch: tiny, ragged and tile-sized
    shapes, every tile width, step counts that leave each remainder."""
    for nx, ny in [(2, 2), (3, 5), (37, 23), (64, 16), (32, 32), (130, 17), (257, 3), (5, 300),
                   (1000, 7), (300, 140)]:
        note("time blocking", storage, nx, ny)
        for blocking in (2, 3):
            for tile in (32, 64, 128):
                a = flb.Lattice(nx, ny, TAU_C1, 1e-3, u0=(0.03, -0.02), seed=4, storage=storage)
                b = flb.Lattice(nx, ny, TAU_C1, 1e-3, u0=(0.03, -0.02), seed=4, storage=storage)
                b.set_time_blocking(blocking, tile)
                assert b.time_blocking() == (blocking, tile)
                a.thermalize()
                b.thermalize()
                for n, t in ((7, 7), (8, 15), (3, 18)):
                    a.step(n)
                    b.step(n)
                    assert a.t == b.t == t
                    assert np.array_equal(a.get_populations(), b.get_populations()), \
                        (nx, ny, blocking, tile, t)


def test_time_blocking_batch_and_graph_periods(flb):
    specs = [dict(nx=70, ny=40, tau=TAU_C1, theta=1e-3, stream_id=0),
             dict(nx=33, ny=129, tau=TAU_C1, theta=1e-3, u0=(0.05, 0.0), stream_id=1),
             dict(nx=8, ny=8, tau=TAU_C1, theta=1e-3, stream_id=2)]
    a = flb.Lattice.batch(specs, seed=6)
    b = flb.Lattice.batch(specs, seed=6)
    b.set_time_blocking(2, 128)
    d = flb.Lattice.batch(specs, seed=6)
    d.set_time_blocking(3, 64)
    # each lattice its own tile in one launch (the size-class form)
    c = flb.Lattice.batch(specs, seed=6)
    c.set_lattice_tiles([32, 64, 32])
    assert c.time_blocking() == (2, 0) and c.lattice_tiles() == [32, 64, 32]
    assert b.lattice_tiles() == [128, 128, 128]
    for h in (a, b, c, d):
        h.thermalize()
        h.run(103, 10)  # graph periods of ten steps plus a ragged tail
        h.run(37, 3)    # odd periods started off-phase
    for i in range(len(specs)):
        for h in (b, c, d):
            assert np.array_equal(a.get_populations(i), h.get_populations(i))
            assert np.array_equal(a.read_correlators(i)[0], h.read_correlators(i)[0])
    with pytest.raises(flb.FlbError):
        b.set_time_blocking(4, 64)
    with pytest.raises(flb.FlbError):
        b.set_time_blocking(2, 256)
    with pytest.raises(flb.FlbError):
        c.set_lattice_tiles([32, 128, 64])
    with pytest.raises(ValueError):
        c.set_lattice_tiles([32, 64])
    assert c.lattice_tiles() == [32, 64, 32]


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_lattice_tiles_equal_one_step_launches(flb, storage):
    """Per-lattice tile shapes on ragged and tiny lattices of one batch give
    the populations of one step per launch, every assignment of the two
    widths to the lattices."""
    sides = [(2, 2), (37, 23), (130, 17), (33, 65), (5, 300)]
    specs = [dict(nx=nx, ny=ny, tau=TAU_C1, theta=1e-3, u0=(0.03, -0.01), stream_id=i)
             for i, (nx, ny) in enumerate(sides)]
    ref = flb.Lattice.batch(specs, seed=9, storage=storage)
    ref.thermalize()
    ref.step(9)
    want = [ref.get_populations(i) for i in range(len(sides))]
    for mask in range(1 << len(sides)):
        tiles = [32 if mask >> i & 1 else 64 for i in range(len(sides))]
        g = flb.Lattice.batch(specs, seed=9, storage=storage)
        g.set_lattice_tiles(tiles)
        g.thermalize()
        g.step(9)
        for i in range(len(sides)):
            assert np.array_equal(g.get_populations(i), want[i]), (tiles, i)
        g.close()


def test_autotune_tiles_per_size_class(flb, tmp_path, monkeypatch):
    """A batch of lattices of several size classes: the whole-path tuner
    (per-class tiles among its candidates) leaves populations, step counter
    and sums unchanged, the run after it has the bits of an untuned handle
    set to the chosen tiles, and a second handle of the same batch takes the
    choice from the cache file."""
    monkeypatch.setenv("FLB_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    sides = [(64, 64), (70, 200), (100, 100), (130, 300), (300, 130), (257, 257), (90, 40),
             (40, 90)]
    specs = [dict(nx=nx, ny=ny, tau=TAU_C1, theta=1e-3, u0=(0.02, 0.0), stream_id=i)
             for i, (nx, ny) in enumerate(sides)]
    ref = flb.Lattice.batch(specs, seed=31)
    g = flb.Lattice.batch(specs, seed=31)
    for h in (ref, g):
        h.thermalize()
        h.step(4)
    cfg, ms = g.autotune_path(4, 5)
    tiles = g.lattice_tiles()
    note("size-class tiles", g.time_blocking(), tiles, ms)
    assert ms > 0 and g.t == 4
    assert all(w in (32, 64, 128) for w in tiles)
    for i in range(len(sides)):
        assert np.array_equal(g.get_populations(i), ref.get_populations(i))
    ref.set_step_config(*cfg)
    if g.time_blocking()[1] == 0:
        ref.set_lattice_tiles(tiles)
    else:
        ref.set_time_blocking(*g.time_blocking())
    for h in (ref, g):
        h.run(20, 5)
    for i in range(len(sides)):
        assert np.array_equal(g.get_populations(i), ref.get_populations(i))
        assert np.array_equal(g.read_correlators(i)[0], ref.read_correlators(i)[0])
    h = flb.Lattice.batch(specs, seed=2)
    cfg2, ms2 = h.autotune_path(4, 5)  # from the cache file
    assert cfg2 == cfg and abs(ms2 - ms) < 1e-5
    assert h.time_blocking() == g.time_blocking() and h.lattice_tiles() == tiles
    assert len((tmp_path / "tune.txt").read_text().splitlines()) == 1


VX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
VY = (0, 0, 1, 0, -1, 1, 1, -1, -1)


def _oracle_site(oracle_lib, f, x, y, t, nx, tau, sigma, seed, stream_id=0):
    """Post-collision values of site (x, y) at time t from the pulled
    populations f[:, y, x] (one site of the oracle's step)."""
    z = oracle_lib.normals_from_words(
        oracle_lib.noise_words(seed, stream_id, t, y * nx + x, 0))
    return oracle_lib.collide_site(np.ascontiguousarray(f[:, y, x]), tau, sigma, z)


@pytest.mark.parametrize("nx,ny", [(4096, 4096), (10900, 10900)])
def test_sampled_sites_at_full_and_maximum_size(flb, oracle_lib, nx, ny):
    """The 4096^2 workload and a lattice at the size limit (populations of
    4.28 GB, just under the 4 GiB reach of the 32-bit offsets), in the launch
    shape the benchmark times: 2000 sampled sites (the corners among them)
    after one step of the one-step kernel and after two steps of the
    two-step kernel, each against the oracle's collision of that site (for
    two steps, of its nine upstream neighbours at t, then of the site at
    t + 1); the two kernels' states after two steps are the same bits, and
    one launch of the three-step kernel gives the bits of three one-step
    launches."""
    c = workloads.CONFIGS["c5_4096"]
    tau, theta, seed = c["tau"], c["theta"], c["seed"]
    sigma = oracle_lib.noise_amplitudes(tau, theta, 1.0)
    note(f"{nx}x{ny} sampled sites")
    kw = dict(u0=c["u0"], seed=seed)
    a = flb.Lattice(nx, ny, tau, theta, **kw)
    a.set_step_config(256, 1, 1)
    a.set_time_blocking(2, 64)
    a.thermalize()
    a.step(4)
    t = a.t
    f0 = a.get_populations()  # f_i(x, t): the pulled values at every site
    b = flb.Lattice(nx, ny, tau, theta, **kw)
    b.set_step_config(256, 1, 1)
    b.set_populations(f0)
    b.t = t
    b.set_time_blocking(1, 64)
    b.step(1)
    f1 = b.get_populations()
    rng = np.random.default_rng(7)
    xs = np.concatenate([[0, nx - 1, 0, nx - 1], rng.integers(0, nx, 1996)])
    ys = np.concatenate([[0, 0, ny - 1, ny - 1], rng.integers(0, ny, 1996)])
    err1 = 0.0
    for x, y in zip(xs.tolist(), ys.tolist()):
        fo = _oracle_site(oracle_lib, f0, x, y, t, nx, tau, sigma, seed)
        got = [f1[i, (y + VY[i]) % ny, (x + VX[i]) % nx] for i in range(9)]
        err1 = max(err1, float(np.abs(np.array(got) - fo).max()))
    del f1
    note("  one step: max |df|", err1)
    assert err1 < 1e-6
    a.step(2)  # one launch of the two-step kernel
    f2 = a.get_populations()
    err2 = 0.0
    for x, y in zip(xs[:500].tolist(), ys[:500].tolist()):
        pulled = np.empty((9, 1, 1))
        for i in range(9):
            xu, yu = (x - VX[i]) % nx, (y - VY[i]) % ny
            pulled[i, 0, 0] = _oracle_site(oracle_lib, f0, xu, yu, t, nx, tau, sigma, seed)[i]
        z = oracle_lib.normals_from_words(oracle_lib.noise_words(seed, 0, t + 1, y * nx + x, 0))
        fo = oracle_lib.collide_site(np.ascontiguousarray(pulled[:, 0, 0]), tau, sigma, z)
        got = [f2[i, (y + VY[i]) % ny, (x + VX[i]) % nx] for i in range(9)]
        err2 = max(err2, float(np.abs(np.array(got) - fo).max()))
    note("  two steps: max |df|", err2)
    assert err2 < 2e-6
    b.step(1)  # second step through the one-step kernel
    assert np.array_equal(b.get_populations(), f2)
    del f2
    # three steps in one launch of the three-step kernel (the shape the
    # benchmark times at 4096^2) against a third one-step launch
    c = flb.Lattice(nx, ny, tau, theta, **kw)
    c.set_step_config(256, 1, 1)
    c.set_populations(f0)
    c.t = t
    c.set_time_blocking(3, 64)
    c.step(3)
    b.step(1)
    assert c.t == b.t == t + 3
    assert np.array_equal(c.get_populations(), b.get_populations())


def test_empty_calls_change_nothing(flb):
    """Zero steps, a run of zero steps, a run without samples, and reading
    the sums before any sample: nothing moves, nothing is counted."""
    a = flb.Lattice(40, 24, TAU_C1, 1e-4, u0=(0.03, 0.0), seed=11)
    a.thermalize()
    f0 = a.get_populations()
    a.step(0)
    a.run(0, 10)
    assert a.t == 0 and np.array_equal(a.get_populations(), f0)
    acc, ns = a.read_correlators()
    assert ns == 0 and not acc.any()
    a.run(25, 0)  # steps only
    b = flb.Lattice(40, 24, TAU_C1, 1e-4, u0=(0.03, 0.0), seed=11)
    b.thermalize()
    b.step(25)
    assert a.t == b.t == 25 and np.array_equal(a.get_populations(), b.get_populations())
    assert a.read_correlators()[1] == 0
    a.accumulate()
    a.step(0)  # a waiting sample stays waiting through no steps
    acc, ns = a.read_correlators()
    assert ns == 1 and acc.any()


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("sides", [[(2311, 1803)], [(2050, 2049)],
                                   [(1000, 2200), (57, 9000), (4100, 901), (56, 58), (3, 2)],
                                   [(66, 65)], [(256, 256)], [(300, 200), (70, 41), (2, 3)],
                                   [(2, 900)], [(513, 500)]])
@pytest.mark.parametrize("theta", [1e-4, 0.0])
def test_library_grouping_equals_one_step_launches(flb, storage, sides, theta):
    """The library's own grouping of the steps (marching launches of four and
    five steps on large lattices, ragged strips and segments; launches of many
    steps on small tiles where the device would be idle) gives the bits of one
    step per launch, for every remainder."""
    note("own grouping", storage, sides, theta)
    specs = [dict(nx=nx, ny=ny, tau=workloads.tau_vector(0.7, 1.1, 0.9), theta=theta,
                  u0=(0.04, -0.02), stream_id=7 + i) for i, (nx, ny) in enumerate(sides)]
    a = flb.Lattice.batch(specs, seed=11, storage=storage)
    b = flb.Lattice.batch(specs, seed=11, storage=storage)
    b.set_time_blocking(1, 64)
    f = workloads.perturbed(a.get_populations()[:, 0, 0], *sides[0], 1e-3, 5)
    for g in (a, b):
        g.thermalize()
        g.set_populations(f)
    for n in (1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 13, 25):
        a.step(n)
        b.step(n)
    for i in range(len(sides)):
        assert np.array_equal(a.get_populations(i), b.get_populations(i)), i


@pytest.mark.parametrize("nx,ny", [(32, 32), (256, 256), (300, 128), (1024, 768)])
@pytest.mark.parametrize("n", [2, 6, 10])
def test_replays_of_captured_steps(flb, nx, ny, n):
    """A caller's graph of an even number of steps advances state and step
    counter as plain calls do at each replay, for every grouping of the steps
    into launches."""
    import torch
    note("captured steps", nx, ny, n)
    g = flb.Lattice(nx, ny, TAU_C1, 1e-3, seed=4)
    ref = flb.Lattice(nx, ny, TAU_C1, 1e-3, seed=4)
    s = torch.cuda.Stream()
    g.set_stream(s)
    for h in (g, ref):
        h.thermalize()
        h.step(n)
        h.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.step(n)
    for replay in range(3):
        with torch.cuda.stream(s):
            graph.replay()
        ref.step(n)
        assert np.array_equal(g.get_populations(), ref.get_populations()), replay
        torch.ones(1000, device="cuda").sum().item()


@pytest.mark.parametrize("nx,ny", [(32, 32), (256, 256), (700, 500), (2048, 2048)])
@pytest.mark.parametrize("calls", [(3, 5), (1, 7), (5, 1), (1, 2, 3, 4)])
def test_replays_of_several_captured_calls(flb, nx, ny, calls):
    """A caller's graph of several calls, an even number of steps in all, with
    plain calls of as many between its replays."""
    import torch
    note("captured calls", nx, ny, calls)
    g = flb.Lattice(nx, ny, TAU_C1, 1e-3, seed=4)
    ref = flb.Lattice(nx, ny, TAU_C1, 1e-3, seed=4)
    with hip_stream(flb) as s:
        g.set_stream(s)
        for h in (g, ref):
            h.thermalize()
            h.step(2)
            h.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            for n in calls:
                g.step(n)
        for replay in range(3):
            with torch.cuda.stream(s):
                graph.replay()
            for n in calls:
                ref.step(n)
            assert np.array_equal(g.get_populations(), ref.get_populations()), replay
            torch.ones(1000, device="cuda").sum().item()
            for h in (g, ref):
                for n in (4, 3, 9):
                    h.step(n)
            assert np.array_equal(g.get_populations(), ref.get_populations()), replay
        g.set_stream(None)
