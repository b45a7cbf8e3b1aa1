"""Performance cases of the library: what its users' programs have it do.

A case is a simulation block: a model is created on the program's own device
buffers, the program steps it K times per pass and looks at the fields (a view
of the buffers on the device, or a copy on the host), and, where it asked for
them, at the per-step reductions.  One case is the batching server with a burst
of mixed requests.  `listed` spans the range from the launch-bound 128^2 grid to
the 32768^2 Cahn-Hilliard grid; `draw` gives more of the same ranges; `exact`
is the same scheme in plain torch / numpy float64.
"""
import functools
import math
from fractions import Fraction

import numpy as np
import torch

import paper_2511_10508_amd as P
from paper_2511_10508_amd.serving import Server

KINDS = {"ac": P.PF_AC, "ch": P.PF_CH, "gs": P.PF_GS, "mc": P.PF_MC, "mh": P.PF_MH}
PARAMS = {"ac": (1.0, 1.0), "ch": (1.0, 1.0), "gs": (0.2, 0.1, 0.04, 0.06), "mc": (1.0, 1.0, 0.5),
          "mh": (1.0, 1.0, 0.5)}
NOISE = {"ac": 0.1, "ch": 0.05, "mc": 0.1, "mh": 0.1}


def _case(kind, n, order, dt, fp, steps, reduce=False, tuned=False, graph=False, host=False,
          spectral=False, direct=False):
    n = list(n) + [1] * (3 - len(n))
    return {"op": "step", "kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "order": order, "dt": dt,
            "fp": fp, "steps": steps, "reduce": reduce, "tuned": tuned, "graph": graph, "host": host,
            "spectral": spectral, "direct": direct}


def listed():
    def named(name, c):
        return dict(c, name=name)
    return [
        # the smallest workload of the benchmark: latency of a small grid, many steps a call
        named("ac2d_128_fp64", _case("ac", (128, 128), 2, 0.05, 64, 1000)),
        # a ragged grid stepped and then plotted: the fields come back to the host
        named("gs2d_515x389_fp32_host", _case("gs", (515, 389), 2, 0.5, 32, 200, graph=True, host=True)),
        # an everyday 2D run, no tuning, no reductions
        named("ch2d_256_fp32", _case("ch", (256, 256), 2, 0.01, 32, 400)),
        # the benchmark's scheme (order 4, mass and energy of every step) at an everyday size
        named("ch2d_1024_fp64_red", _case("ch", (1024, 1024), 4, 0.01, 64, 100, reduce=True)),
        # two coupled fields at a middling size, created and stepped with the defaults
        named("mc2d_2048_fp32", _case("mc", (2048, 2048), 4, 0.01, 32, 50)),
        # the benchmark's headline workload, autotuned as a production run is
        named("ch2d_32768_fp64_red_tuned", _case("ch", (32768, 32768), 4, 0.01, 64, 8, reduce=True, tuned=True)),
        # small 3D run with the reductions of every step
        named("ch3d_96_fp32_red", _case("ch", (96, 96, 96), 2, 0.005, 32, 50, reduce=True)),
        # large 3D reaction-diffusion, autotuned
        named("gs3d_512_fp64_tuned", _case("gs", (512, 512, 512), 2, 0.5, 64, 8, tuned=True)),
        # the 3D precision-study workload (order 4), autotuned
        named("ch3d_384_fp64_red_tuned", _case("ch", (384, 384, 384), 4, 0.005, 64, 8, reduce=True, tuned=True)),
        # Model H on a box with unequal sides
        named("mh3d_256x192x160_fp64", _case("mh", (256, 192, 160), 4, 0.005, 64, 10)),
        # the semi-implicit Fourier step
        named("spectral_ch2d_2048_fp64", _case("ch", (2048, 2048), 2, 0.5, 64, 20, spectral=True)),
        # a burst of mixed requests through the batching server, results fetched
        {"name": "serve_24", "op": "serve", "requests": 24, "max2d": 512, "max3d": 96, "max_steps": 800},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["small2d", "small2d", "mid2d", "mid2d", "large2d", "small3d", "large3d", "mh",
                         "spectral", "row", "direct", "serve"])
    fp = rng.choice([64, 32])
    if family == "small2d":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        n = (_log(rng, 64, 640), _log(rng, 64, 640))
        if rng.random() < 0.5:
            n = tuple(max(64, v // 32 * 32) for v in n)
        return _case(kind, n, rng.choice([2, 4]), _dt(kind), fp, _log(rng, 100, 1000),
                     graph=rng.random() < 0.3, host=rng.random() < 0.3, reduce=rng.random() < 0.3)
    if family == "mid2d":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        n = (_log(rng, 640, 4096), _log(rng, 640, 4096))
        return _case(kind, n, rng.choice([2, 4, 6]), _dt(kind), fp, _log(rng, 20, 100),
                     reduce=rng.random() < 0.5, tuned=rng.random() < 0.3)
    if family == "large2d":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        n = (_log(rng, 4096, 20000), _log(rng, 4096, 20000))
        return _case(kind, n, rng.choice([2, 4]), _dt(kind), fp, 8, reduce=rng.random() < 0.5, tuned=True)
    if family == "small3d":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        n = tuple(_log(rng, 32, 160) for _ in range(3))
        return _case(kind, n, rng.choice([2, 4]), _dt(kind) / 2, fp, _log(rng, 20, 100),
                     reduce=rng.random() < 0.5)
    if family == "large3d":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        n = tuple(_log(rng, 192, 448) for _ in range(3))
        return _case(kind, n, rng.choice([2, 4, 6]), _dt(kind) / 2, fp, 8, reduce=rng.random() < 0.5, tuned=True)
    if family == "mh":
        if rng.random() < 0.5:
            return _case("mh", (_log(rng, 256, 3000), _log(rng, 256, 3000)), rng.choice([2, 4]), 0.005, fp, 20)
        return _case("mh", tuple(_log(rng, 64, 300) for _ in range(3)), rng.choice([2, 4]), 0.004, fp, 8)
    if family == "spectral":
        kind = rng.choice(["ac", "ch"])
        sides = [256, 384, 500, 512, 729, 1000, 1024, 1536, 2048, 2187, 3000, 4096]
        if rng.random() < 0.7:
            return _case(kind, (rng.choice(sides), rng.choice(sides)), 2, 0.5, fp, _log(rng, 10, 30),
                         spectral=True)
        n = tuple(rng.choice([64, 96, 100, 125, 128, 192, 256]) for _ in range(3))
        return _case(kind, n, 2, 0.5, fp, 10, spectral=True)
    if family == "row":
        kind = rng.choice(["ac", "ch", "gs", "mc"])
        return _case(kind, (_log(rng, 10000, 1 << 24),), rng.choice([2, 4]), _dt(kind), fp, 50,
                     reduce=rng.random() < 0.5)
    if family == "direct":
        if rng.random() < 0.5:
            return _case("ch", (_log(rng, 512, 8192), _log(rng, 512, 8192)), rng.choice([2, 4]), 0.01, fp, 10,
                         direct=True, reduce=True)
        return _case("ch", tuple(_log(rng, 64, 320) for _ in range(3)), rng.choice([2, 4]), 0.004, fp, 10,
                     direct=True, reduce=True)
    return {"op": "serve", "requests": rng.randint(8, 24), "max2d": _log(rng, 200, 512),
            "max3d": _log(rng, 48, 96), "max_steps": _log(rng, 200, 800)}


def _dt(kind):
    return {"ac": 0.05, "ch": 0.01, "gs": 0.4, "mc": 0.01}[kind]


# ---------------------------------------------------------------- inputs --
def _ndim(c):
    return 3 if c["nz"] > 1 else 2 if c["ny"] > 1 else 1


def _nfields(c):
    return 1 + _ndim(c) if c["kind"] == "mh" else 2 if c["kind"] in ("gs", "mc") else 1


def _initial(c, seed, f):
    """Field f of the initial state, (nz, ny, nx) on the GPU in the storage
    type: noise about zero, or for Gray-Scott a state u = 1, v = 0 with seeded
    patches u = 0.5, v = 0.25, and noise."""
    dtype = torch.float64 if c["fp"] == 64 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed % (1 << 40)) + 17 * f)
    shape = (c["nz"], c["ny"], c["nx"])
    x = torch.rand(shape, generator=g, dtype=dtype, device="cuda")
    if c["kind"] != "gs":
        a = NOISE[c["kind"]]
        return x.mul_(2 * a).sub_(a)
    x.mul_(0.02).sub_(0.01).add_(1.0 if f == 0 else 0.0)
    rng = np.random.default_rng(seed)
    for _ in range(20):
        at = [int(rng.integers(0, max(1, n - 15))) for n in shape]
        x[at[0]:at[0] + 16, at[1]:at[1] + 16, at[2]:at[2] + 16] += -0.5 if f == 0 else 0.25
    return x


def _desc(c):
    n = (c["nx"], c["ny"], c["nz"])[:_ndim(c)]
    flags = ((P.PF_REDUCE_EACH_STEP if c["reduce"] else 0) | (P.PF_USE_GRAPH if c["graph"] else 0) |
             (P.PF_SPECTRAL if c["spectral"] else 0) | (P.PF_BIHARMONIC_DIRECT if c["direct"] else 0))
    return P.make_desc(KINDS[c["kind"]], n, dx=1.0, dt=c["dt"], order=c["order"],
                       precision=P.PF_FP64 if c["fp"] == 64 else P.PF_FP32, params=PARAMS[c["kind"]],
                       flags=flags)


def _requests(c, seed):
    """A burst of the serving workload: models, sides, orders, parameters and
    step counts mixed, FP32 storage."""
    rng = np.random.default_rng(seed)
    out = []
    # the sizes and step counts are those of the case, the seed shapes values only, so
    # that every seed is the same amount of work
    mix = np.random.default_rng(505)
    for i in range(c["requests"]):
        kind = ("ac", "ch", "gs")[int(mix.integers(0, 3))]
        ndim = 2 + int(mix.integers(0, 2))
        side = int(round(math.exp(mix.uniform(math.log(64 if ndim == 2 else 32),
                                              math.log(c["max2d"] if ndim == 2 else c["max3d"])))))
        steps = int(round(math.exp(mix.uniform(math.log(100), math.log(c["max_steps"])))))
        order = (2, 4)[int(mix.integers(0, 2))]
        jit = rng.uniform(0.9, 1.1, size=4)
        params = [p * j for p, j in zip(PARAMS[kind], jit)]
        dt = {"ac": 0.05, "ch": 0.008, "gs": 0.4}[kind] * (0.5 if ndim == 3 else 1.0)
        out.append({"kind": kind, "ndim": ndim, "side": side, "steps": steps, "order": order,
                    "params": params, "dt": dt, "seed": int(rng.integers(1, 1 << 40)), "cube": max(2, side // 32)})
    return out


# what a program creates once: one stream (its simulations run one after another), one server
@functools.lru_cache(maxsize=None)
def _stream():
    return torch.cuda.Stream()


@functools.lru_cache(maxsize=None)
def _server():
    return Server(hbm_budget=8 << 30, max_slots=64)


def prepare(case, seed):
    if case["op"] == "serve":
        reqs = _requests(case, seed)
        calls = []
        for r in reqs:
            d = P.make_desc(KINDS[r["kind"]], (r["side"],) * r["ndim"], dx=1.0, dt=r["dt"], order=r["order"],
                            precision=P.PF_FP32, params=r["params"])
            if r["kind"] == "gs":
                ic, icp = P.PF_IC_GS_CUBES, (20, r["cube"], 0.01)
            else:
                ic, icp = P.PF_IC_UNIFORM, (-NOISE[r["kind"]], NOISE[r["kind"]])
            calls.append((d, ic, r["seed"], icp, r["steps"], (r["side"],) * r["ndim"], 2 if r["kind"] == "gs" else 1))
        return {"server": _server(), "calls": calls}
    d = _desc(case)
    nf = _nfields(case)
    pitch = P.buffer_elems(d) // (case["ny"] * case["nz"])
    dtype = torch.float64 if case["fp"] == 64 else torch.float32
    bufs = [torch.zeros((case["nz"], case["ny"], pitch), dtype=dtype, device="cuda") for _ in range(2 * nf)]
    for f in range(nf):
        bufs[2 * f][..., :case["nx"]] = _initial(case, seed, f)
    torch.cuda.synchronize()
    m = P.Model(d, stream=_stream().cuda_stream, bufs=[b.data_ptr() for b in bufs])
    if case["tuned"]:
        m.autotune()
    return {"model": m, "case": case, "bufs": bufs}


def run(state):
    if "server" in state:
        srv, calls = state["server"], state["calls"]
        tickets = [srv.submit(*call[:5]) for call in calls]
        srv.drain()
        done = {r["ticket"]: r for r in srv.poll()}
        out = []
        for t, call in zip(tickets, calls):
            out.append({"fields": [srv.fetch(t, f, call[5]) for f in range(call[6])],
                        "steps": done[t]["steps_done"]})
            srv.release(t)
        return out
    m, c, bufs = state["model"], state["case"], state["bufs"]
    m.step(c["steps"])
    out = {}
    if c["reduce"]:
        hi, lo = m.reduce_history(P.PF_RED_MASS0, c["steps"])
        out["mass"] = hi + lo
        if c["kind"] in ("ac", "ch"):
            hi, lo = m.reduce_history(P.PF_RED_ENERGY, c["steps"])
            out["energy"] = hi + lo
    fields = []
    for f in range(_nfields(c)):
        if c["host"]:
            fields.append(m.get_field(f))
        else:
            at = m.field_device(f)[0]
            fields.append(next(b for b in bufs[2 * f:2 * f + 2] if b.data_ptr() == at)[..., :c["nx"]])
    out["fields"] = fields
    return out


# ------------------------------------------------------------------ work --
def _site_flops(kind, ndim, order, direct):
    """Operations of one site-step: an r-point second derivative per axis is
    r (2 adds, a subtraction, a multiply-add) on the neighbour pairs."""
    r = order // 2
    lap = r * (2 * ndim + 3)
    first = 3 * r
    if direct:
        return lap * ndim + (r + 1) * (2 * ndim + 3) + 8
    return {"ac": lap + 5, "ch": 2 * lap + 6, "gs": 2 * lap + 12, "mc": 2 * lap + 10,
            "mh": (2 + ndim) * lap + 2 * ndim * (first + 3) + 6}[kind]


def work(case):
    if case["op"] == "serve":
        b = f = 0.0
        for r in _requests(case, 0):
            nf, sites = (2 if r["kind"] == "gs" else 1), r["side"] ** r["ndim"]
            b += sites * nf * 8  # FP64 results on the host
            f += sites * r["steps"] * _site_flops(r["kind"], r["ndim"], r["order"], False)
        return {"bytes": b, "flops": f}
    sites = case["nx"] * case["ny"] * case["nz"]
    # every field is read once and written once a pass
    b = 2.0 * _nfields(case) * sites * (case["fp"] // 8)
    if case["spectral"]:
        # two real transforms, the local term and the implicit update per step
        f = case["steps"] * sites * (2 * 2.5 * math.log2(sites) + 4 + 12)
    else:
        f = float(case["steps"]) * sites * _site_flops(case["kind"], _ndim(case), case["order"], case["direct"])
    return {"bytes": b, "flops": f}


# ----------------------------------------------------------------- exact --
@functools.lru_cache(maxsize=None)
def _weights(order, deriv):
    """Centred weights of the deriv-th derivative (even: w_-j = w_j, first:
    w_-j = -w_j), accuracy `order`, solved in exact rationals."""
    m = order // 2 + (1 if deriv == 4 else 0)
    par = deriv % 2
    n = m if par else m + 1
    a = [[Fraction(j) ** (2 * i + par) for j in range(par, m + 1)] for i in range(n)]
    b = [Fraction(math.factorial(deriv), 2) if 2 * i + par == deriv else Fraction(0) for i in range(n)]
    if not par:
        for row in a:
            row[0] /= 2  # j = 0 counts once
    for i in range(n):  # Gauss-Jordan
        p = next(k for k in range(i, n) if a[k][i] != 0)
        a[i], a[p], b[i], b[p] = a[p], a[i], b[p], b[i]
        s = a[i][i]
        a[i], b[i] = [v / s for v in a[i]], b[i] / s
        for k in range(n):
            if k != i and a[k][i] != 0:
                s = a[k][i]
                a[k], b[k] = [v - s * w for v, w in zip(a[k], a[i])], b[k] - s * b[i]
    return ([0.0] if par else []) + [float(v) for v in b]


def _axes(ndim):
    return [2, 1, 0][:ndim]  # x, y, z of a (z, y, x) array


def _second(u, w, axis):
    out = torch.zeros_like(u)
    for j in range(1, len(w)):
        out.add_(torch.roll(u, j, axis).add_(torch.roll(u, -j, axis)).sub_(u, alpha=2.0), alpha=w[j])
    return out


def _first(u, w, axis):
    out = torch.zeros_like(u)
    for j in range(1, len(w)):
        out.add_(torch.roll(u, -j, axis).sub_(torch.roll(u, j, axis)), alpha=w[j])
    return out


def _lap(u, w, ndim):
    out = _second(u, w, _axes(ndim)[0])
    for ax in _axes(ndim)[1:]:
        out.add_(_second(u, w, ax))
    return out


def _advance(kind, ndim, order, dt, params, s, direct=False):
    """One forward-Euler step of the fields s (float64), dx = 1."""
    w = _weights(order, 2)
    if kind == "ac":
        u, = s
        return [u + dt * (_lap(u, w, ndim) + params[0] * u - params[1] * u ** 3)]
    if kind == "ch":
        u, = s
        g = params[1] * u ** 3 - params[0] * u
        if not direct:
            return [u.add(_lap(g.sub_(_lap(u, w, ndim)), w, ndim), alpha=dt)]
        w4, ax = _weights(order, 4), _axes(ndim)
        rhs = _lap(g, w, ndim)
        for i, a in enumerate(ax):
            rhs.sub_(_second(u, w4, a))  # the difference form of any even stencil
            for b in ax[i + 1:]:
                rhs.sub_(_second(_second(u, w, a), w, b), alpha=2.0)
        return [u + dt * rhs]
    if kind == "gs":
        u, v = s
        uvv = u * v * v
        return [u + dt * (params[0] * _lap(u, w, ndim) - uvv + params[2] * (1 - u)),
                v + dt * (params[1] * _lap(v, w, ndim) + uvv - (params[2] + params[3]) * v)]
    if kind == "mc":
        p, r = s
        return [p + dt * (_lap(p, w, ndim) + params[0] * p - params[1] * p ** 3 - 2 * p * r),
                r + dt * _lap(r + params[2] * p * p, w, ndim)]
    w1, m, js = _weights(order, 1), s[0], s[1:]
    mu = params[1] * m ** 3 - params[0] * m - _lap(m, w, ndim)
    div = torch.zeros_like(m)
    for j, a in zip(js, _axes(ndim)):
        div.add_(_first(m * j, w1, a))
    out = [m + dt * (_lap(mu, w, ndim) - params[2] * div)]
    for j, a in zip(js, _axes(ndim)):
        out.append(j + dt * (_lap(j, w, ndim) + params[2] * m * _first(mu, w1, a)))
    return out


def _spectral_steps(c, u):
    k = [torch.fft.fftfreq(n, d=1.0 / (2 * math.pi), dtype=torch.float64, device=u.device)
         for n in (c["nz"], c["ny"])]
    kx = torch.fft.rfftfreq(c["nx"], d=1.0 / (2 * math.pi), dtype=torch.float64, device=u.device)
    k2 = k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + kx[None, None, :] ** 2
    dt, (c1, c2), dims = c["dt"], PARAMS[c["kind"]], (0, 1, 2)
    for _ in range(c["steps"]):
        local = torch.fft.rfftn(c2 * u ** 3 - c1 * u, dim=dims)
        uh = torch.fft.rfftn(u, dim=dims)
        if c["kind"] == "ac":
            uh = (uh - dt * local) / (1 + dt * k2)
        else:
            uh = (uh - dt * k2 * local) / (1 + dt * k2 * k2)
        u = torch.fft.irfftn(uh, s=u.shape, dim=dims)
    return u


_M64 = (1 << 64) - 1
_GOLD = 0x9E3779B97F4A7C15


def _mix(z):
    """SplitMix64's finaliser on numpy uint64 values."""
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _uniform(seed, stream, idx):
    with np.errstate(over="ignore"):
        key = _mix(np.array([(seed + (stream + 1) * _GOLD) & _M64], dtype=np.uint64))
        z = _mix(key + (idx.astype(np.uint64) + np.uint64(1)) * np.uint64(_GOLD))
    return (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


def _served_initial(r):
    """The initial state that the server documents for a request, rounded to FP32."""
    shape = (1,) * (3 - r["ndim"]) + (r["side"],) * r["ndim"]
    idx = np.arange(int(np.prod(shape)))
    a = 0.01 if r["kind"] == "gs" else NOISE[r["kind"]]
    s = [(-a + 2 * a * _uniform(r["seed"], f, idx)).reshape(shape) for f in range(2 if r["kind"] == "gs" else 1)]
    if r["kind"] == "gs":
        corner = _uniform(r["seed"], 2, np.arange(60)).reshape(20, 3)
        inside = np.zeros(shape, dtype=bool)
        z, y, x = np.meshgrid(*[np.arange(n) for n in shape], indexing="ij")
        for cx, cy, cz in corner:
            at = [min(int(v * n), n - 1) for v, n in zip((cz, cy, cx), shape)]
            inside |= (((z - at[0]) % shape[0] < min(r["cube"], shape[0])) &
                       ((y - at[1]) % shape[1] < min(r["cube"], shape[1])) &
                       ((x - at[2]) % shape[2] < min(r["cube"], shape[2])))
        s = [np.where(inside, 0.5, 1.0) + s[0], np.where(inside, 0.25, 0.0) + s[1]]
    return [torch.from_numpy(v.astype(np.float32).astype(np.float64)).cuda() for v in s]


def exact(case, seed):
    if case["op"] == "serve":
        out = []
        for r in _requests(case, seed):
            s = _served_initial(r)
            for _ in range(r["steps"]):
                s = _advance(r["kind"], r["ndim"], r["order"], r["dt"], r["params"], s)
            out.append({"fields": [v.reshape((r["side"],) * r["ndim"]) for v in s], "steps": r["steps"]})
        return out
    ndim, out = _ndim(case), {}
    s = [_initial(case, seed, f).double() for f in range(_nfields(case))]
    if case["spectral"]:
        return {"fields": [_spectral_steps(case, s[0])]}
    p, w, mass, energy = PARAMS[case["kind"]], _weights(case["order"], 2), [], []
    for _ in range(case["steps"]):
        if case["reduce"]:
            mass.append(s[0].sum())
            if case["kind"] in ("ac", "ch"):
                u = s[0]
                energy.append((_lap(u, w, ndim).mul_(-0.5).add_(u ** 3, alpha=p[1] / 4)
                               .sub_(u, alpha=p[0] / 2).mul_(u)).sum())
        s = _advance(case["kind"], ndim, case["order"], case["dt"], p, s, case["direct"])
    if mass:
        out["mass"] = torch.stack(mass)
    if energy:
        out["energy"] = torch.stack(energy)
    out["fields"] = s
    return out
