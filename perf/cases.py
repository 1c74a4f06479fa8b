"""Performance cases of the library: what its users run, call by call.

Two kinds of calls are covered, on D2Q9 lattices (``Lattice``) and on the
other velocity sets (``DqLattice``):

* sampling runs: ``run(steps, every)`` followed by a read of the correlators
  of every lattice, the way a measurement ends;
* restarts: a saved state and its time are put back (``set_populations``,
  ``t``), the lattice steps on, and the new state is read.

``listed()`` holds the workloads of ``workloads.py``, of the tests and of the
benchmark, with the number of steps per read cut so that a pass stays short;
``draw()`` gives others of the same ranges.  The library computes in FP32
(and stores in FP32 or 16 bits), so results are handed on as FP32.

``exact()`` is the method itself in FP64 with torch: the Philox stream and the
normals as flb.h documents them, the moment tables by Gram-Schmidt, Eqs. (1)
to (12) as written.
"""
import math

import numpy as np
import torch

import paper_1010_1233_amd as flb

THETA = 1e-4

# Velocity sets: dimension, velocities, weights, the polynomials that are
# orthonormalised into the moments.
_D2Q9 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0),
         (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
_D3Q15 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)] + \
    [(-1 if c & 1 else 1, -1 if c & 2 else 1, -1 if c & 4 else 1) for c in range(8)]
SETS = {
    "D1Q3": (1, [(0, 0, 0), (1, 0, 0), (-1, 0, 0)], [2 / 3, 1 / 6, 1 / 6],
             lambda x, y, z, q: [1 + 0 * x, x, x * x - 1 / 3]),
    "D2Q9": (2, _D2Q9, [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4,
             lambda x, y, z, q: [1 + 0 * x, x, y, x * x - y * y, x * y, q - 2 / 3, x * q, y * q,
                                 q * q]),
    "D3Q15": (3, _D3Q15, [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8,
              lambda x, y, z, q: [1 + 0 * x, x, y, z, 3 * x * x - q, y * y - z * z, x * y, y * z,
                                  z * x, q - 1, x * q, y * q, z * q, x * y * z, q * q]),
}


def listed():
    base = dict(storage="f32", moments=False, ladd=False, tau=0.8, ux=0.0, tune=False)
    d2 = dict(base, model="D2Q9", lattices=1, uneven=False, restart=False)
    dq = dict(base, lattices=1, uneven=False, restart=False, ny=1, nz=1)
    return [
        # the paper's own regime: an ensemble of 20 x 20 lattices at tau = 1,
        # all nine moments, a sample after every step
        dict(d2, name="paper_ensemble_20", nx=20, ny=20, nz=1, lattices=512, tau=1.0,
             moments=True, steps=200, every=1),
        # the smallest single lattice: launches and latency
        dict(d2, name="single_32", nx=32, ny=32, nz=1, steps=1000, every=10),
        # an ordinary single lattice, far too small to fill the GPU
        dict(d2, name="single_256", nx=256, ny=256, nz=1, steps=1000, every=10),
        # the large lattice of the benchmark, launch shape tuned once
        dict(d2, name="large_4096", nx=4096, ny=4096, nz=1, tau=0.6, ux=0.05, steps=2000,
             every=10, tune=True),
        # the Galilean-invariance sweep: six mean velocities, four realisations each
        dict(d2, name="galilean_24x512", nx=512, ny=512, nz=1, lattices=24, ux=0.2, steps=1000,
             every=10),
        # lattices of uneven sides and relaxation times in one batch
        dict(d2, name="uneven_64", nx=1024, ny=64, nz=1, lattices=64, uneven=True, ux=0.1,
             steps=500, every=10),
        # 16-bit storage, sampled
        dict(d2, name="bf16_2048", nx=2048, ny=2048, nz=1, tau=0.6, ux=0.05, storage="bf16",
             steps=500, every=10),
        # resume from a checkpoint on a lattice of ragged sides, 16-bit storage
        dict(d2, name="restart_f16_1001x700", nx=1001, ny=700, nz=1, storage="f16", restart=True,
             steps=200, every=0),
        # three dimensions: a small cube sampled often, a box with unequal
        # sides, and a large cube stepped between checkpoints
        dict(dq, name="d3q15_32", model="D3Q15", nx=32, ny=32, nz=32, steps=200, every=10),
        dict(dq, name="d3q15_160x96x60", model="D3Q15", nx=160, ny=96, nz=60, steps=100, every=10),
        dict(dq, name="d3q15_restart_192", model="D3Q15", nx=192, ny=192, nz=192, restart=True,
             steps=200, every=0),
        # one dimension, a long line between checkpoints
        dict(dq, name="d1q3_restart_4m", model="D1Q3", nx=1 << 22, restart=True, steps=500,
             every=0),
    ]


def _log(rng, lo, hi):
    """A whole number, spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["ensemble", "single", "single", "batch", "uneven", "restart", "d3", "d3",
                         "d3 restart", "d1"])
    c = dict(model="D2Q9", storage="f32", moments=False, ladd=False, ux=0.0, tune=False, lattices=1,
             uneven=False, restart=False, nz=1, tau=round(rng.uniform(0.55, 1.5), 3), every=10)
    if family == "ensemble":
        n = rng.choice([16, 20, 24, rng.randint(8, 32)])
        c.update(nx=n, ny=n if rng.random() < 0.6 else rng.randint(8, 32),
                 lattices=_log(rng, 64, 1024), moments=rng.random() < 0.5, ladd=rng.random() < 0.3,
                 ux=rng.choice([0.0, 0.05, 0.1]), steps=rng.randint(50, 200),
                 every=rng.choice([1, 1, 2, 10]))
    elif family == "single":
        sides = [_log(rng, 20, 2048) for _ in range(2)]
        if rng.random() < 0.5:
            sides = [1 << max(4, s.bit_length() - 1) for s in sides]
        sites = sides[0] * sides[1]
        c.update(nx=sides[0], ny=sides[1], ux=rng.choice([0.0, 0.05]),
                 storage=rng.choice(["f32", "f32", "bf16", "f16"]), tune=rng.random() < 0.2,
                 moments=sites < 400000 and rng.random() < 0.3,
                 steps=rng.randint(20, 100) * (10 if sites < 1000000 else 4))
    elif family == "batch":
        n = rng.choice([64, 128, 256, 512, rng.randint(40, 600)])
        c.update(nx=n, ny=n, lattices=max(2, min(64, (6 << 20) // (n * n))),
                 ux=rng.choice([0.05, 0.1, 0.2]), steps=rng.randint(20, 60) * 10)
    elif family == "uneven":
        lo = _log(rng, 16, 128)
        c.update(nx=lo * rng.choice([4, 8]), ny=lo, lattices=rng.randint(8, 48), uneven=True,
                 ux=0.1, steps=rng.randint(10, 40) * 10)
    elif family == "restart":
        c.update(nx=_log(rng, 24, 2000), ny=_log(rng, 24, 2000), restart=True,
                 storage=rng.choice(["f32", "bf16", "f16"]), ux=rng.choice([0.0, 0.1]),
                 ladd=rng.random() < 0.2, steps=rng.randint(20, 400), every=0)
    elif family == "d3":
        c.update(model="D3Q15", nx=_log(rng, 6, 160), ny=_log(rng, 6, 80), nz=_log(rng, 6, 60),
                 ladd=rng.random() < 0.3, steps=rng.randint(5, 20) * 10)
    elif family == "d3 restart":
        c.update(model="D3Q15", nx=_log(rng, 6, 180), ny=_log(rng, 6, 180), nz=_log(rng, 6, 180),
                 restart=True, steps=rng.randint(20, 200), every=0)
    elif rng.random() < 0.5:
        c.update(model="D1Q3", nx=_log(rng, 64, 2000), ny=1, steps=rng.randint(20, 100) * 10)
    else:
        c.update(model="D1Q3", nx=_log(rng, 64, 1 << 22), ny=1, restart=True,
                 steps=rng.randint(50, 500), every=0)
    return c


# ---------------------------------------------------------------------------
# Parameters of a case's lattices
# ---------------------------------------------------------------------------
def _specs(case):
    """One dict per lattice: sides, relaxation times per moment, mean
    velocity, stream id."""
    D, v, _, _ = SETS[case["model"]]
    Q, out = len(v), []
    rng = np.random.default_rng(4)
    for i in range(case["lattices"]):
        nx, ny, shear, ux = case["nx"], case["ny"], case["tau"], case["ux"]
        if case["uneven"]:  # sides between ny and nx, log-uniform
            nx, ny = (int(round(math.exp(rng.uniform(math.log(case["ny"]), math.log(case["nx"])))))
                      for _ in range(2))
            shear, ux = float(rng.uniform(0.55, 1.5)), float(rng.uniform(0.0, case["ux"]))
        elif case["lattices"] > 1 and ux:  # a sweep of mean velocities
            ux = ux * (i % 6) / 5
        tau = [1.0] * Q
        for a in range(D + 1, D + D * (D + 1) // 2):  # the shear modes (bulk and ghosts: 1)
            tau[a] = shear
        if D == 1:
            tau[2] = shear
        out.append(dict(nx=nx, ny=ny, nz=case["nz"], tau=tau, theta=THETA, rho0=1.0,
                        u0=(ux, 0.0), stream_id=i))
    return out


def _state(case, seed):
    """A saved state of the first lattice: equilibrium plus fluctuations of
    the thermal size, and the time it was saved at."""
    D, v, w, _ = SETS[case["model"]]
    v, w = np.array(v, float), np.array(w)
    s = _specs(case)[0]
    u = np.array([s["u0"][0], 0.0, 0.0])
    vu, V = v @ u, s["nx"] * s["ny"] * s["nz"]
    f0 = w * (1 + 3 * vu + 4.5 * vu * vu - 1.5 * (u @ u))
    gen = torch.Generator(device=_device()).manual_seed(seed)
    f = torch.randn(len(w), V, generator=gen, device=_device(), dtype=torch.float32).double()
    f *= torch.tensor(np.sqrt(3 * THETA * w), device=f.device)[:, None]
    f += torch.tensor(f0, device=f.device)[:, None]
    shape = (s["ny"], s["nx"]) if case["model"] == "D2Q9" else (s["nz"], s["ny"], s["nx"])
    return f.cpu().numpy().reshape((len(w),) + shape), 1000


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ---------------------------------------------------------------------------
# The calls
# ---------------------------------------------------------------------------
def prepare(case, seed):
    specs = _specs(case)
    if case["model"] == "D2Q9":
        g = flb.Lattice.batch(specs, seed=seed, storage=case["storage"], ladd=case["ladd"],
                              moments=case["moments"])
    else:
        D, s = SETS[case["model"]][0], specs[0]
        g = flb.DqLattice(case["model"], (s["nx"], s["ny"], s["nz"])[:D], s["tau"], s["theta"],
                          u0=(s["u0"][0], 0.0, 0.0)[:D], seed=seed, ladd=case["ladd"])
    state = dict(case=case, g=g)
    if case["restart"]:
        state["f"], state["t"] = _state(case, seed)
        state["out"] = torch.empty(state["f"].shape, dtype=torch.float32)
    else:
        g.thermalize()
        if case["tune"]:
            g.autotune_path(10, case["every"])
        sizes = [g.nkinds * s["ny"] * s["nz"] * (s["nx"] // 2 + 1) for s in specs]
        state["out"] = torch.empty(sum(sizes), dtype=torch.float32)
        state["parts"] = torch.split(state["out"], sizes)
    return state


def run(state):
    case, g, out = state["case"], state["g"], state["out"]
    if case["restart"]:
        g.set_populations(state["f"])
        if case["model"] == "D2Q9":
            g.t = state["t"]
        g.step(case["steps"])
        out.copy_(torch.from_numpy(g.get_populations()))
        return out
    g.run(case["steps"], case["every"])
    for i, part in enumerate(state["parts"]):
        if case["model"] == "D2Q9":
            sums, _ = g.read_normalized_raw(i)
        else:
            sums, _ = g.read_correlators()
        part.copy_(torch.from_numpy(sums).view(-1))
    return out


def work(case):
    """Bytes: the state read and written once, the results written once (FP64,
    and a restart's state read as FP64).  Flops: per site update the collision
    and its noise, per sample the transforms of the fields along each axis and
    the FP64 products."""
    D, v, _, _ = SETS[case["model"]]
    Q, b, f = len(v), 0, 0
    noise = -(-(Q - D - 1) // 6)
    cell = 4 if case["storage"] == "f32" else 2
    fields = 1 + 2 * D + (Q - D - 1 if case["moments"] or case["model"] != "D2Q9" else 0)
    for s in _specs(case):
        V = s["nx"] * s["ny"] * s["nz"]
        k = (s["nx"] // 2 + 1) * s["ny"] * s["nz"]
        b += 2 * cell * Q * V
        f += case["steps"] * V * (10 * Q + 100 * noise)
        if case["restart"]:
            b += 2 * 8 * Q * V
        else:
            samples = case["steps"] // case["every"]
            kinds = fields + (10 if case["model"] == "D2Q9" else 2 if D > 1 else 0)
            b += 8 * kinds * k
            f += samples * (fields * 2.5 * V * math.log2(max(2, V)) + 4 * kinds * k)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The method in FP64
# ---------------------------------------------------------------------------
def _tables(model):
    D, v, w, poly = SETS[model]
    v, w = np.array(v, float), np.array(w)
    x, y, z = v.T
    m = []
    for h in poly(x, y, z, x * x + y * y + z * z):
        for r in m:
            h = h - (w * h) @ r * r
        m.append(h / math.sqrt((w * h) @ h))
    return D, v, w, np.array(m)


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    mask = 0xFFFFFFFF
    k0, k1 = seed & mask, (seed >> 32) & mask
    zero = torch.zeros_like(c0)
    c = [c0, zero + c1, c2, zero + c3]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # the low 64 bits: all of the product
        c = [((p1 >> 32) & mask) ^ c[1] ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k1, p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _normals(site, t, stream, count, seed):
    """`count` unit normals per site, in sixes per draw."""
    z = []
    for d in range(-(-count // 6)):
        w = _philox(site, t, stream, d, seed)
        for p in range(3):
            r = (2 * (w[p] >> 9) + 1).double() * 2.0 ** -24
            al = ((w[p] & 0x1FF) << 10) | ((w[3] >> (10 * p)) & 0x3FF)
            a = (2 * al + 1).double() * (2 * math.pi * 2.0 ** -20)
            rad = torch.sqrt(-2 * torch.log(r))
            z += [rad * torch.cos(a), rad * torch.sin(a)]
    return torch.stack(z[:count])


def exact(case, seed):
    specs, model = _specs(case), case["model"]
    sizes = [s["nx"] * s["ny"] * s["nz"] for s in specs]
    updates = sum(sizes) * case["steps"]
    if updates > 1e10 or (not torch.cuda.is_available() and updates > 2e7):
        return None  # over about 20 seconds
    dev = _device()
    D, v, w, m = _tables(model)
    Q = len(w)
    T = lambda a: torch.tensor(np.asarray(a, dtype=float), device=dev)  # noqa: E731
    tw, tv, tm, back = T(w)[:, None], T(v), T(m), T((w * m).T.copy())
    # every lattice's sites in one array; src[i]: the site that streams along v_i into each
    site, lat, src, off = [], [], [], 0
    for i, s in enumerate(specs):
        n = torch.arange(sizes[i], device=dev)
        x, y, z = n % s["nx"], n // s["nx"] % s["ny"], n // (s["nx"] * s["ny"])
        src.append(torch.stack([off + (x - int(c[0])) % s["nx"] + s["nx"] *
                                ((y - int(c[1])) % s["ny"] + s["ny"] * ((z - int(c[2])) % s["nz"]))
                                for c in v]))
        site.append(n)
        lat.append(torch.full_like(n, i))
        off += sizes[i]
    site, lat, src = torch.cat(site), torch.cat(lat), torch.cat(src, 1)
    stream = torch.tensor([s["stream_id"] for s in specs], device=dev)[lat]
    one = len(specs) == 1 or not (case["uneven"] or case["ux"])
    pick = (lambda a: T(a[0]).reshape(-1, 1)) if one else (lambda a: T(a).T[:, lat].contiguous())
    mu = 3 * THETA
    tau = np.array([s["tau"] for s in specs])
    sigma = np.sqrt(mu * (2 * tau - 1)) / tau
    if case["ladd"]:
        sigma[:, 1 + D + D * (D + 1) // 2:] = 0
    rate, amp = pick(1 / tau[:, D + 1:]), pick(sigma[:, D + 1:])
    u0 = pick(np.array([[s["u0"][0]] + [0.0] * (D - 1) for s in specs]))

    def equilibrium(rho, u):
        vu = tv[:, :D] @ u
        return tw * rho * (1 + 3 * vu + 4.5 * vu * vu - 1.5 * (u * u).sum(0))

    t = 0
    if case["restart"]:
        f, t = _state(case, seed)
        f = torch.tensor(f.reshape(Q, -1), device=dev)
    else:
        add = torch.sqrt(mu * tw) * _normals(site, 0xFFFFFFFF, stream, Q, seed)
        at = 0
        for n in sizes:
            add[:, at:at + n] -= add[:, at:at + n].mean(1, keepdim=True)
            at += n
        f = equilibrium(torch.ones_like(site, dtype=torch.float64), u0.expand(D, len(site))) + add
        del add
    if case["restart"] and model != "D2Q9":
        t = 0  # the other velocity sets have no call that sets the time: a first pass starts at 0
    sums, samples = [0.0] * len(specs), 0
    for _ in range(case["steps"]):
        rho, j = f.sum(0), tv.T[:D] @ f
        M = tm[D + 1:] @ f
        M0 = tm[D + 1:] @ equilibrium(rho, j / rho)
        M0[D * (D + 1) // 2:] = 0
        dM = (M0 - M) * rate + amp * _normals(site, t, stream, Q - D - 1, seed)
        f = f + back[:, D + 1:] @ dM
        f = torch.gather(f, 1, src)
        t += 1
        if case["every"] and t % case["every"] == 0:
            samples += 1
            rho, j = f.sum(0), tv.T[:D] @ f
            X = torch.cat([rho[None] - 1, j - u0, j / rho - u0, tm[D + 1:] @ f])
            at = 0
            for i, s in enumerate(specs):
                F = torch.fft.rfftn(X[:, at:at + sizes[i]].reshape(-1, s["nz"], s["ny"], s["nx"]),
                                    dim=(1, 2, 3))
                sums[i] = sums[i] + _kinds(F, D, model == "D2Q9", case["moments"])
                at += sizes[i]
    if case["restart"]:
        s = specs[0]
        return f.reshape((Q, s["ny"], s["nx"]) if model == "D2Q9" else
                         (Q, s["nz"], s["ny"], s["nx"])).cpu()
    out = []
    for s, n, a in zip(specs, sizes, sums):
        a[:, 0, 0, 0] = 0
        if model == "D2Q9":
            cs = 1 / math.sqrt(3)
            norm = [1 / (n * mu)] + [1 / (n * THETA)] * 6 + [1 / (n * mu * cs)] * 8 + \
                [1 / (n * mu)] * 6
            a = a / samples * T(norm)[:len(a), None, None, None]
        out.append(a.reshape(-1))
    return torch.cat(out).cpu()


def _kinds(F, D, d2q9, moments):
    """The products of one sample's spectra, in the library's order."""
    sq = (F.conj() * F).real
    auto = [sq[:1 + 2 * D]]
    if d2q9:
        pairs = [(3, 4), (0, 1), (0, 2), (0, 3), (0, 4)]
    else:
        pairs = [(1 + D, 2 + D)] if D > 1 else []
    for a, b in pairs:
        c = F[a] * F[b].conj()
        auto += [c.real[None], c.imag[None]]
    if moments or not d2q9:
        auto.append(sq[1 + 2 * D:])
    return torch.cat(auto)
