"""Performance cases: what a user of this library has it do.

Each case is a dict of plain values; ``prepare`` makes the inputs a program
holds before the call (on the GPU, from a seed), ``run`` is one pass through
the public entry points, ``work`` the bytes and flops the pass cannot do
without, ``exact`` its result from plain torch in 64 bits.

Kinds:
  sweep    a fixed number of Jacobi sweeps, one, two or three per pass over
           memory, with the residual of every ``every``-th iterate fused into
           the passes (the time-stepping use of jacobi3d_sweep*)
  solve    poisson_solve from a zero guess, plain FP64 or mixed precision
  batch    jacobi3d_sweep_batch over uneven grids
  serve    a burst of requests through a Poisson server, results on the host
  jacobi2d the 2D Laplace iteration of jacobi2d_sweeps
  pw       one momentum advection tendency
  tracer   a number of donor-cell tracer steps
  reduce   sum or dot_product of long vectors
"""
import math

import numpy as np
import torch

from paper_2409_18824_amd import j3d


def listed():
    return [
        # the smallest call: one sweep of a 64^3 grid and the residual that
        # goes with it, as a program with its own iteration control makes it
        {"name": "sweep_f64_64", "kind": "sweep", "dtype": "f64", "nx": 64, "ny": 64, "nz": 64,
         "per_pass": 1, "sweeps": 1, "every": 1},
        # the benchmark's grid and pass kind: 512^3 FP64, three sweeps per
        # pass, residual every 10 sweeps (30 of its 500 sweeps)
        {"name": "sweeps_f64_512", "kind": "sweep", "dtype": "f64", "nx": 512, "ny": 512, "nz": 512,
         "per_pass": 3, "sweeps": 30, "every": 10},
        # FP32 relaxation on a ragged, cache-sized grid, two sweeps per pass
        {"name": "sweeps_f32_333x222x111", "kind": "sweep", "dtype": "f32", "nx": 333, "ny": 222, "nz": 111,
         "per_pass": 2, "sweeps": 10, "every": 0},
        # the small solve: 64^3, 100 sweeps, residual history of every sweep
        {"name": "solve_f64_64_every", "kind": "solve", "mode": "fp64", "nx": 64, "ny": 64, "nz": 64,
         "sweeps": 100, "every": 1},
        # an ordinary solve on a ragged grid that fits the last-level cache
        {"name": "solve_f64_181x143x160", "kind": "solve", "mode": "fp64", "nx": 181, "ny": 143, "nz": 160,
         "sweeps": 200, "every": 10},
        # mixed precision at the size of the mixed benchmark's default run
        {"name": "solve_mixed_256", "kind": "solve", "mode": "mixed", "nx": 256, "ny": 256, "nz": 256,
         "sweeps": 200, "every": 50},
        # uneven grids of the batch benchmark's sizes (32..256 per axis)
        {"name": "batch_40", "kind": "batch", "grids": 40, "lo": 32, "hi": 256, "sweeps": 60, "every": 10},
        # a burst of requests of the serving benchmark's smaller sizes, with
        # right-hand sides from and solutions to the host
        {"name": "serve_12", "kind": "serve", "requests": 12, "lo": 32, "hi": 96, "sweeps": 500},
        # the 2D jacobi benchmark's grid, a fiftieth of its iterations
        {"name": "jacobi2d_1024", "kind": "jacobi2d", "nx": 1024, "ny": 1024, "sweeps": 2000},
        # multi-field stencils at the tracer benchmark's shape
        {"name": "pw_1024x512x512", "kind": "pw", "nx": 1024, "ny": 512, "nz": 512},
        {"name": "tracer_1024x512x512", "kind": "tracer", "nx": 1024, "ny": 512, "nz": 512, "steps": 20},
        # dot_product at the reduction benchmark's length
        {"name": "dot_2p27", "kind": "reduce", "op": "dot", "n": 1 << 27},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "solve", "solve", "batch", "serve", "jacobi2d", "pw", "tracer", "reduce"])
    c = {"kind": kind}
    if kind == "sweep":
        c.update(dtype=rng.choice(["f64", "f64", "f32"]), nx=_log_int(rng, 32, 512), ny=_log_int(rng, 32, 512),
                 nz=_log_int(rng, 32, 512), per_pass=rng.choice([1, 2, 3]))
        c["sweeps"] = c["per_pass"] * rng.randint(1, 10)
        c["every"] = 10 if c["dtype"] == "f64" and rng.random() < 0.7 else 0
    elif kind == "solve":
        c.update(mode=rng.choice(["fp64", "mixed"]), nx=_log_int(rng, 32, 320), ny=_log_int(rng, 32, 320),
                 nz=_log_int(rng, 32, 320))
        c["every"] = 50 if c["mode"] == "mixed" else rng.choice([1, 10, 50])
        c["sweeps"] = 50 * rng.randint(1, 4)
    elif kind == "batch":
        lo = rng.randint(32, 96)
        c.update(grids=rng.randint(4, 48), lo=lo, hi=rng.randint(lo, 224), sweeps=10 * rng.randint(2, 6), every=10)
    elif kind == "serve":
        lo = rng.randint(32, 64)
        c.update(requests=rng.randint(4, 12), lo=lo, hi=rng.randint(lo, 96), sweeps=50 * rng.randint(4, 10))
    elif kind == "jacobi2d":
        c.update(nx=_log_int(rng, 64, 2048), ny=_log_int(rng, 64, 2048), sweeps=_log_int(rng, 50, 2000))
    elif kind == "pw":
        c.update(nx=_log_int(rng, 64, 1024), ny=_log_int(rng, 64, 512), nz=_log_int(rng, 64, 512))
    elif kind == "tracer":
        c.update(nx=_log_int(rng, 64, 1024), ny=_log_int(rng, 64, 512), nz=_log_int(rng, 64, 512),
                 steps=rng.randint(1, 20))
    else:
        c.update(op=rng.choice(["sum", "dot"]), n=_log_int(rng, 1 << 10, 1 << 27))
    return c


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------

_DT = {"f64": (j3d.F64, torch.float64), "f32": (j3d.F32, torch.float32)}


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _interior(g, shape, lo, hi, halo, dtype=torch.float64):
    """Padded tensor (z, y, x): interior uniform on [lo, hi), halo constant."""
    a = torch.full([n + 2 for n in shape], halo, dtype=dtype, device="cuda")
    inner = a[tuple(slice(1, -1) for _ in shape)]
    inner.copy_(torch.rand(shape, generator=g, dtype=dtype, device="cuda").mul_(hi - lo).add_(lo))
    return a


def _h(*dims):
    return 1.0 / (max(dims) + 1)


def _sweep_inputs(case, seed):
    g, dt = _gen(seed), _DT[case["dtype"]][1]
    shape = (case["nz"], case["ny"], case["nx"])
    return _interior(g, shape, 0.0, 1.0, 0.0, dt), _interior(g, shape, -1.0, 1.0, 0.0, dt)


def _solve_input(case, seed):
    return _interior(_gen(seed), (case["nz"], case["ny"], case["nx"]), -1.0, 1.0, 0.0)


def _batch_shapes(case):
    """The grids' extents (x, y, z): fixed by the case, not by the seed."""
    r = np.random.default_rng(case["grids"] * 1000003 + case["lo"] * 1009 + case["hi"])
    return [tuple(int(v) for v in r.integers(case["lo"], case["hi"] + 1, 3)) for _ in range(case["grids"])]


def _batch_inputs(case, seed):
    g = _gen(seed)
    return [_interior(g, d[::-1], -1.0, 1.0, 0.0) for d in _batch_shapes(case)]


def _serve_sizes(case):
    r = np.random.default_rng(case["requests"] * 1000003 + case["lo"] * 1009 + case["hi"])
    u = r.random(case["requests"])
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** float(v))) for v in u]


def _serve_inputs(case, seed):
    r = np.random.default_rng(int(seed) * 7919 + 17)
    out = []
    for n in _serve_sizes(case):
        f = np.zeros((n + 2, n + 2, n + 2))
        f[1:-1, 1:-1, 1:-1] = r.random((n, n, n)) * 2.0 - 1.0
        out.append(f)
    return out


def _jacobi2d_input(case, seed):
    """Random interior, the benchmark's boundary: top edge 1, other edges 0."""
    u = _interior(_gen(seed), (case["ny"], case["nx"]), 0.0, 1.0, 0.0)
    u[-1, :] = 1.0
    return u


def _pw_inputs(case, seed):
    g = _gen(seed)
    return [_interior(g, (case["nz"], case["ny"], case["nx"]), -1.0, 1.0, 0.25) for _ in range(3)]


def _tracer_inputs(case, seed):
    """t, u, v, w, r: a tracer in [0, 1), transports small enough for stable steps."""
    g = _gen(seed)
    shape = (case["nz"], case["ny"], case["nx"])
    t = _interior(g, shape, 0.0, 1.0, 0.5)
    q = [_interior(g, shape, -0.1, 0.1, 0.0) for _ in range(3)]
    return [t] + q + [_interior(g, shape, 0.5, 1.5, 1.0)]


def _reduce_inputs(case, seed):
    g = _gen(seed)
    k = 2 if case["op"] == "dot" else 1
    return [torch.rand(case["n"], generator=g, dtype=torch.float64, device="cuda") for _ in range(k)]


def _farray(t):
    """A library array with the layout FArray.empty gives, holding tensor t."""
    code = j3d.F32 if t.dtype == torch.float32 else j3d.F64
    nz, ny, nx = (n - 2 for n in t.shape)
    a = j3d.FArray.empty(nx, ny, nz, dtype=code)
    a.view().copy_(t)
    return a


def _like(a):
    nx, ny, nz = a.interior
    return j3d.FArray.empty(nx, ny, nz, dtype=a.dtype)


class _Served:
    """A server with the requests a client is about to send it."""

    def __init__(self, case, seed):
        self.f = _serve_inputs(case, seed)
        self.u = [np.zeros_like(f) for f in self.f]
        self.sweeps = case["sweeps"]
        self.server = j3d.Server(hbm_budget_bytes=8 << 30, max_slots=64, cycle_sweeps=50)

    def __del__(self):
        if getattr(self, "server", None) is not None:
            self.server.close()


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "sweep":
        u, f = _sweep_inputs(case, seed)
        s["h"] = _h(case["nx"], case["ny"], case["nz"])
        s["u"], s["f"] = _farray(u), _farray(f)
        s["w"] = [_like(s["u"]), _like(s["u"])]
        n = len(_resid_points(case))
        s["res"] = torch.zeros(max(n, 1), dtype=torch.float64, device="cuda")
    elif kind == "solve":
        s["h"] = _h(case["nx"], case["ny"], case["nz"])
        s["f"] = _farray(_solve_input(case, seed))
        s["u"] = _like(s["f"])
    elif kind == "batch":
        s["grids"] = []
        for d, f in zip(_batch_shapes(case), _batch_inputs(case, seed)):
            ff = _farray(f)
            s["grids"].append((_like(ff), _like(ff), ff, _h(*d)))
        s["res"] = torch.zeros(case["grids"] * (case["sweeps"] // case["every"] + 1), dtype=torch.float64,
                               device="cuda")
    elif kind == "serve":
        s["served"] = _Served(case, seed)
    elif kind == "jacobi2d":
        u = _jacobi2d_input(case, seed)
        s["h"] = _h(case["nx"], case["ny"])
        s["u"] = []
        for _ in range(2):
            a = j3d.FArray.empty2d(case["nx"], case["ny"])
            a.view()[0].copy_(u)
            s["u"].append(a)
        s["res"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    elif kind == "pw":
        s["in"] = [_farray(t) for t in _pw_inputs(case, seed)]
        s["out"] = [_like(s["in"][0]) for _ in range(3)]
    elif kind == "tracer":
        fields = _tracer_inputs(case, seed)
        s["t0"] = _farray(fields[0])
        s["t"] = [_farray(fields[0]), _farray(fields[0])]
        s["in"] = [_farray(t) for t in fields[1:]]
    else:
        s["x"] = _reduce_inputs(case, seed)
        s["res"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    return s


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------

def _resid_points(case):
    """Iterates whose residual norm a sweep case reports."""
    e = case["every"]
    return [] if e == 0 else [k for k in range(0, case["sweeps"] + 1) if k % e == 0 and (k < case["sweeps"] or k > 1)]


_SWEEP = {1: j3d.jacobi3d_sweep, 2: j3d.jacobi3d_sweep2, 3: j3d.jacobi3d_sweep3}


def _run_sweep(s):
    c, h, f, res = s["case"], s["h"], s["f"], s["res"]
    P, S, E = c["per_pass"], c["sweeps"], c["every"]
    step = _SWEEP[P]
    cur, q = s["u"], 0
    for i, at in enumerate(range(0, S, P)):
        out = s["w"][i % 2]
        # the stage of this pass that forms a reported iterate (every is even
        # with two-sweep passes, which report their input's residual only)
        stage = next((o for o in range(P) if E and (at + o) % E == 0), None)
        if stage is None:
            step(cur, out, f, h)
        elif P == 3:
            step(cur, out, f, h, resid_out=res[q:q + 1], resid_after=stage)
            q += 1
        else:
            step(cur, out, f, h, resid_out=res[q:q + 1])
            q += 1
        cur = out
    if E and S > 1 and S % E == 0:
        j3d.residual_l2(cur, f, h, out=res[q:q + 1])
    return {"u": cur.view()} if not E else {"u": cur.view(), "resid": res}


def _run_solve(s):
    c = s["case"]
    j3d.j3d_fill_const(s["u"], 0.0)
    if c["mode"] == "mixed":
        r = j3d.poisson_solve(s["u"], s["f"], s["h"], mode=j3d.MODE_MIXED, rtol=1e-10, max_sweeps=c["sweeps"],
                              inner_sweeps=c["every"], history_cap=c["sweeps"] + 1)
    else:
        r = j3d.poisson_solve(s["u"], s["f"], s["h"], rtol=1e-10, max_sweeps=c["sweeps"], check_every=c["every"],
                              history_cap=c["sweeps"] + 1)
    return {"u": s["u"].view(), "history": r.history, "norm_f": r.norm_f, "resid": r.resid, "sweeps": r.sweeps}


def _run_served(sv):
    srv = sv.server
    order = {}
    for k, (f, u) in enumerate(zip(sv.f, sv.u)):
        n = f.shape[0] - 2
        order[srv.submit(n, 1.0 / (n + 1), 1e-10, sv.sweeps, f_host=f, u_out=u)] = k
    srv.drain()
    resid, sweeps = np.zeros(len(order)), np.zeros(len(order), dtype=np.int64)
    for r in srv.poll(len(order)):
        resid[order[r["ticket"]]] = r["resid"]
        sweeps[order[r["ticket"]]] = r["sweeps"]
    return {"u": sv.u, "resid": resid, "sweeps": sweeps}


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "sweep":
        return _run_sweep(s)
    if kind == "solve":
        return _run_solve(s)
    if kind == "batch":
        j3d.jacobi3d_sweep_batch(s["grids"], c["sweeps"], c["every"], s["res"])
        return {"u": [g[c["sweeps"] % 2].view() for g in s["grids"]], "resid": s["res"]}
    if kind == "serve":
        return _run_served(s["served"])
    if kind == "jacobi2d":
        j3d.jacobi2d_sweeps(s["u"][0], s["u"][1], c["sweeps"], s["h"], resid_out=s["res"])
        return {"u": s["u"][c["sweeps"] % 2].view(), "resid": s["res"]}
    if kind == "pw":
        d = 1.0 / 1024
        j3d.pw_advection(*s["in"], *s["out"], d, d, d)
        return [a.view() for a in s["out"]]
    if kind == "tracer":
        s["t"][0].storage.copy_(s["t0"].storage)  # a run starts from its initial tracer
        j3d.tracer_advection(s["t"][0], s["t"][1], *s["in"], c["steps"])
        return s["t"][c["steps"] % 2].view()
    if c["op"] == "dot":
        j3d.j3d_dot(s["x"][0], s["x"][1], out=s["res"])
    else:
        j3d.j3d_sum(s["x"][0], out=s["res"])
    return s["res"]


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; 8 flops per Jacobi update."""
    kind = case["kind"]
    if kind == "sweep":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 3.0 * n * (8 if case["dtype"] == "f64" else 4), "flops": 8.0 * n * case["sweeps"]}
    if kind == "solve":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 16.0 * n, "flops": 8.0 * n * case["sweeps"]}
    if kind == "batch":
        n = sum(a * b * c for a, b, c in _batch_shapes(case))
        return {"bytes": 24.0 * n, "flops": 8.0 * n * case["sweeps"]}
    if kind == "serve":
        n = sum(a ** 3 for a in _serve_sizes(case))
        return {"bytes": 16.0 * n, "flops": 8.0 * n * case["sweeps"]}
    if kind == "jacobi2d":
        n = case["nx"] * case["ny"]
        return {"bytes": 16.0 * n, "flops": 4.0 * n * case["sweeps"]}
    if kind == "pw":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 48.0 * n, "flops": 60.0 * n}
    if kind == "tracer":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 48.0 * n, "flops": 25.0 * n * case["steps"]}
    return {"bytes": 8.0 * case["n"] * (2 if case["op"] == "dot" else 1), "flops": float(case["n"])}


# ----------------------------------------------------------------------------
# The same results from plain torch in 64 bits
# ----------------------------------------------------------------------------

def _neighbours(u):
    s = u[1:-1, 1:-1, :-2] + u[1:-1, 1:-1, 2:]
    s += u[1:-1, :-2, 1:-1]
    s += u[1:-1, 2:, 1:-1]
    s += u[:-2, 1:-1, 1:-1]
    s += u[2:, 1:-1, 1:-1]
    return s


def _jacobi_exact(u, f, h, sweeps, points=()):
    """u after `sweeps` FP64 sweeps, and the residual norms of the iterates in points."""
    u, hf = u.clone(), f[1:-1, 1:-1, 1:-1] * (h * h)
    res = []
    for k in range(sweeps + 1):
        if k in points:
            r = f[1:-1, 1:-1, 1:-1] - (6.0 * u[1:-1, 1:-1, 1:-1] - _neighbours(u)) / (h * h)
            res.append(math.sqrt(float(torch.sum(r * r))))
        if k < sweeps:
            s = _neighbours(u)
            s += hf
            u[1:-1, 1:-1, 1:-1] = s / 6.0
    return u, res


def _exact_sweep(case, seed):
    u, f = _sweep_inputs(case, seed)
    pts = set(_resid_points(case))
    h = _h(case["nx"], case["ny"], case["nz"])
    out, res = _jacobi_exact(u.double(), f.double(), h, case["sweeps"], pts)
    if not case["every"]:
        return {"u": out}
    want = torch.zeros(max(len(_resid_points(case)), 1), dtype=torch.float64)
    want[:len(res)] = torch.tensor(res, dtype=torch.float64)
    return {"u": out, "resid": want}


def _exact_solve(case, seed):
    # a correction cycle is the same sweeps in exact arithmetic: the plain
    # iteration is the 64-bit result of both modes
    f = _solve_input(case, seed)
    S, e = case["sweeps"], case["every"]
    pts = set(range(0, S + 1, e)) | {S}
    u, res = _jacobi_exact(torch.zeros_like(f), f, _h(case["nx"], case["ny"], case["nz"]), S, pts)
    return {"u": u, "history": np.array(res[: S // e + 1]), "norm_f": math.sqrt(float(torch.sum(f * f))), "resid": res[-1],
            "sweeps": S}


def _exact_batch(case, seed):
    us, rows = [], []
    pts = set(range(0, case["sweeps"] + 1, case["every"]))
    for d, f in zip(_batch_shapes(case), _batch_inputs(case, seed)):
        u, res = _jacobi_exact(torch.zeros_like(f), f, _h(*d), case["sweeps"], pts)
        us.append(u)
        rows += res
    return {"u": us, "resid": torch.tensor(rows, dtype=torch.float64)}


def _exact_serve(case, seed):
    us, res = [], []
    for f in _serve_inputs(case, seed):
        n = f.shape[0] - 2
        u, r = _jacobi_exact(torch.zeros(f.shape, dtype=torch.float64, device="cuda"), torch.from_numpy(f).cuda(),
                             1.0 / (n + 1), case["sweeps"], {case["sweeps"]})
        us.append(u.cpu().numpy())
        res.append(r[0])
    return {"u": us, "resid": np.array(res), "sweeps": np.full(len(res), case["sweeps"], dtype=np.int64)}


def _exact_jacobi2d(case, seed):
    u, h = _jacobi2d_input(case, seed), _h(case["nx"], case["ny"])

    def nb():
        s = u[1:-1, :-2] + u[1:-1, 2:]
        s += u[:-2, 1:-1]
        s += u[2:, 1:-1]
        return s

    for _ in range(case["sweeps"]):
        u[1:-1, 1:-1] = nb() / 4.0
    r = (nb() - 4.0 * u[1:-1, 1:-1]) / (h * h)
    return {"u": u[None], "resid": torch.sqrt(torch.sum(r * r)).reshape(1)}


def _exact_pw(case, seed):
    """Centred flux form: minus the divergence of the momentum flux."""
    q = _pw_inputs(case, seed)
    c = 0.25 * 1024
    inner = (slice(1, -1),) * 3

    def at(a, *shifts):  # the field at interior points shifted by (x, y, z) steps
        d = [0, 0, 0]
        for axis, n in shifts:
            d[axis] += n
        sl = [slice(1 + d[ax], a.shape[2 - ax] - 1 + d[ax]) for ax in (2, 1, 0)]
        return a[tuple(sl)]

    out = []
    for m in range(3):  # component on its own face, staggered along axis m
        tend = None
        for ax in range(3):
            qa = q[ax]
            if ax == m:
                sm = at(q[m], (ax, -1)) + at(q[m])
                sp = at(q[m]) + at(q[m], (ax, 1))
                d = (sm * sm - sp * sp) * c
            else:
                lo = (at(qa, (ax, -1)) + at(qa, (ax, -1), (m, 1))) * (at(q[m], (ax, -1)) + at(q[m]))
                hi = (at(qa) + at(qa, (m, 1))) * (at(q[m]) + at(q[m], (ax, 1)))
                d = (lo - hi) * c
            tend = d if tend is None else tend + d
        full = torch.zeros_like(q[m])
        full[inner] = tend
        out.append(full)
    return out


def _exact_tracer(case, seed):
    t, u, v, w, r = _tracer_inputs(case, seed)
    i = (slice(1, -1),) * 3
    lo = {2: (slice(1, -1), slice(1, -1), slice(0, -2)), 1: (slice(1, -1), slice(0, -2), slice(1, -1)),
          0: (slice(0, -2), slice(1, -1), slice(1, -1))}
    hi = {2: (slice(1, -1), slice(1, -1), slice(2, None)), 1: (slice(1, -1), slice(2, None), slice(1, -1)),
          0: (slice(2, None), slice(1, -1), slice(1, -1))}
    for _ in range(case["steps"]):
        div = None
        for ax, q in ((2, u), (1, v), (0, w)):
            up = q[i].clamp(min=0.0) * t[i] + q[i].clamp(max=0.0) * t[hi[ax]]
            dn = q[lo[ax]].clamp(min=0.0) * t[lo[ax]] + q[lo[ax]].clamp(max=0.0) * t[i]
            up -= dn
            div = up if div is None else div.add_(up)
        t[i] -= r[i] * div
    return t


def exact(case, seed):
    kind = case["kind"]
    if kind == "reduce":
        x = _reduce_inputs(case, seed)
        p = x[0] * x[1] if case["op"] == "dot" else x[0]
        return torch.tensor([math.fsum(p.cpu().numpy())], dtype=torch.float64)
    return {"sweep": _exact_sweep, "solve": _exact_solve, "batch": _exact_batch, "serve": _exact_serve,
            "jacobi2d": _exact_jacobi2d, "pw": _exact_pw, "tracer": _exact_tracer}[kind](case, seed)
