"""Performance cases of the library: the work its users have it do, through
the public Python entry points (`Lattice`, `Pool`), over the range of sizes,
storage types and options the library takes.

Kinds of case:
  frame  one resident lattice: advance it by some steps, then read the density
         and velocity fields on the device (a time-marching run that looks at
         a frame every so often);
  pool   many resident lattices of uneven size: advance them together by one
         batched call, then read the fields of the jobs that are finished;
  job    a whole run from host arrays: initial fields in, steps, populations
         out to host memory.

Single-precision lattices hand their fields on in float32, double-precision
ones in float64.
"""
import math
import random

import numpy as np
import torch

import paper_0707_2437_amd as lbm

ESIZE = {"f64": 8, "f32": 4, "f32s": 4, "f16s": 2}
# Most lattice-site updates of one drawn case of a kind (the largest listed ones do as many).
MOST_FRAME = 8192 * 8192 * 20
MOST_POOL = 9_000_000_000
FLOPS = 90  # of Eq. 5 with Eqs. 2 and 3, per site and step


def _frame(name, nx, ny, dtype, steps, tau=0.6, c2=0.2, init="wave", model="forcing", field=False, inlet=False):
    return {"name": name, "kind": "frame", "nx": nx, "ny": ny, "dtype": dtype, "steps": steps, "tau": tau, "c2": c2,
            "init": init, "model": model, "field": field, "inlet": inlet}


def _pool(name, count, lo, hi, law, dtype, mode, steps, sizes, every, uneven):
    return {"name": name, "kind": "pool", "count": count, "lo": lo, "hi": hi, "law": law, "dtype": dtype,
            "mode": mode, "steps": steps, "sizes": sizes, "every": every, "uneven": uneven}


def listed():
    return [
        # The smallest call: one step of a small ragged lattice and a look at it (an interactive run, a
        # coupled code that exchanges fields every step).
        _frame("frame_397x131_f32", 397, 131, "f32", 1, init="pulse"),
        # The parity set-up of the sound wave on a small square lattice: many steps of almost no work.
        _frame("wave_64x64_f64", 64, 64, "f64", 1000, tau=0.8),
        # The paper's progressive waves: one wavelength on a lattice four sites high, for thousands of steps.
        _frame("channel_4000x4_f64", 4000, 4, "f64", 2000, tau=0.53, c2=0.04),
        # The paper's sound-speed experiment: a channel driven by an oscillating inlet density, one period.
        _frame("inlet_2400x4_f64", 2400, 4, "f64", 500, inlet=True),
        # An acoustic lens that changes between calls (c^2 varying in space and time): ragged, odd step count.
        _frame("lens_1000x777_f32", 1000, 777, "f32", 101, field=True, init="pulse"),
        # The headline: a large plane sound wave, in single and in double precision.
        _frame("wave_4096x4096_f32", 4096, 4096, "f32", 20),
        _frame("wave_4096x4096_f64", 4096, 4096, "f64", 20),
        # Shifted storage: the altered-equilibrium model on a ragged lattice in single precision, and the
        # largest lattice of the range in half precision.
        _frame("equilibrium_4099x2731_f32s", 4099, 2731, "f32s", 25, tau=0.7, c2=0.25, model="equilibrium"),
        _frame("shear_8192x8192_f16s", 8192, 8192, "f16s", 20, tau=0.7, c2=0.25, init="shear"),
        # A batch of independent lattices of uneven size, tau and c^2 taken through a whole run by one call.
        _pool("batch_32_f32_graph", 32, 64, 1024, "uniform", "f32", "graph", 1000, 1, 1, False),
        # One tick of a job server: jobs of many sizes advance together, the finished ones are read out.
        _pool("tick_24_f32_grouped", 24, 128, 2048, "log", "f32", "grouped", 100, 2, 8, True),
        # A run from host arrays to host arrays (a checkpoint in, a checkpoint out).
        {"name": "job_1024x1024_f64", "kind": "job", "nx": 1024, "ny": 1024, "dtype": "f64", "steps": 100,
         "tau": 0.6, "c2": 0.2, "init": "wave"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    tau, c2 = round(rng.uniform(0.55, 1.5), 3), round(rng.uniform(0.04, 0.55), 3)
    kind = rng.choice(["frame", "frame", "frame", "frame", "pool", "pool", "job"])
    if kind == "frame":
        dtype = rng.choice(["f64", "f32", "f32", "f32s", "f16s"])
        init = rng.choice(["wave", "shear", "pulse"])
        option = rng.choice(["", "", "", "field", "inlet", "equilibrium"])
        nx = _log_int(rng, 48, 8192)
        ny = _log_int(rng, 4, 8192)
        steps = _log_int(rng, 1, 2000)
        # a large lattice is stepped less often per look, and half precision is for large ones
        steps = max(1, min(steps, MOST_FRAME // (nx * ny * ESIZE[dtype] // 2)))
        return {"kind": kind, "nx": nx, "ny": ny, "dtype": dtype, "steps": steps, "tau": tau, "c2": c2, "init": init,
                "model": "equilibrium" if option == "equilibrium" else "forcing", "field": option == "field",
                "inlet": option == "inlet"}
    if kind == "pool":
        dtype = rng.choice(["f32", "f32", "f32s", "f64"])
        law = rng.choice(["uniform", "log"])
        count = _log_int(rng, 4, 64)
        hi = _log_int(rng, 128, 1024)
        lo = max(64, hi // rng.choice([2, 8, 16]))
        steps = _log_int(rng, 20, 1000)
        steps = max(2, min(steps, MOST_POOL // (count * hi * hi * ESIZE[dtype] // 4)))
        return {"kind": kind, "count": count, "lo": lo, "hi": hi, "law": law, "dtype": dtype,
                "mode": rng.choice(["grouped", "graph", "persistent"]), "steps": steps,
                "sizes": rng.randrange(1 << 20), "every": rng.choice([4, 8]), "uneven": rng.random() < 0.5}
    side = _log_int(rng, 64, 1024)
    return {"kind": "job", "nx": side, "ny": max(8, min(1024, side * rng.choice([1, 2, 3]) // 2)),
            "dtype": "f64", "steps": _log_int(rng, 10, 200), "tau": tau, "c2": c2,
            "init": rng.choice(["wave", "shear", "pulse"])}


# ---------------------------------------------------------------------------
# Inputs


def _fields(nx, ny, c2, init, gen):
    """Initial (rho, ux, uy) on the device, float64, with a phase or centre from the seed."""
    u = lambda: float(torch.rand((), generator=gen, dtype=torch.float64, device="cuda"))  # noqa: E731
    x = torch.arange(nx, dtype=torch.float64, device="cuda")[None, :]
    y = torch.arange(ny, dtype=torch.float64, device="cuda")[:, None]
    rho = torch.ones(ny, nx, dtype=torch.float64, device="cuda")
    ux, uy = torch.zeros_like(rho), torch.zeros_like(rho)
    if init == "wave":  # plane sound wave of amplitude 1e-3 and density noise of 1e-4
        s = 1e-3 * torch.sin(2 * math.pi * (x / nx + u()))
        rho += s + 1e-4 * (2 * torch.rand(ny, nx, generator=gen, dtype=torch.float64, device="cuda") - 1)
        ux += math.sqrt(c2) * s
    elif init == "shear":  # shear wave
        ux += 0.01 * torch.sin(2 * math.pi * (y / ny + u()))
    else:  # Gaussian density pulse, amplitude up to the nonlinear onset
        amp, sigma = 0.01 + 0.09 * u(), max(min(nx, ny) / 16.0, 1.0)
        cx, cy = nx * (0.25 + 0.5 * u()), ny * (0.25 + 0.5 * u())
        rho += amp * torch.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (2 * sigma * sigma))
    return rho, ux, uy


def _lens(nx, ny, c2):
    """c^2 halved in the middle of the lattice (an acoustic lens)."""
    x = torch.arange(nx, dtype=torch.float64, device="cuda")[None, :]
    y = torch.arange(ny, dtype=torch.float64, device="cuda")[:, None]
    s = min(nx, ny) / 6.0
    return (c2 * (1 - 0.5 * torch.exp(-((x - nx / 2) ** 2 + (y - ny / 2) ** 2) / (2 * s * s)))).contiguous()


INLET = (1e-3, 500.0)  # amplitude and period of the inlet density


def _pool_specs(case):
    r = random.Random(case["sizes"])

    def side():
        if case["law"] == "log":
            return int(round(2 ** r.uniform(math.log2(case["lo"]), math.log2(case["hi"]))))
        return r.randint(case["lo"], case["hi"])

    specs = []
    for k in range(case["count"]):
        nx = side()
        ny = nx if case["law"] == "log" else side()
        done = k % case["every"] == 0  # the jobs that finish in this call
        steps = r.randint(1, case["steps"]) if case["uneven"] and done else case["steps"]
        specs.append({"nx": nx, "ny": ny, "tau": r.uniform(0.55, 1.5), "c2": r.uniform(0.04, 0.55), "done": done,
                      "steps": steps})
    return specs


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def prepare(case, seed):
    gen = _gen(seed)
    if case["kind"] == "frame":
        nx, ny = case["nx"], case["ny"]
        model = lbm.MODEL_EQUILIBRIUM if case["model"] == "equilibrium" else lbm.MODEL_FORCING
        L = lbm.Lattice(nx, ny, case["tau"], case["c2"], case["dtype"], model=model)
        L.set_stream(torch.cuda.current_stream())
        lens = None
        if case["field"]:
            lens = _lens(nx, ny, case["c2"])
            L.set_c2_field_device(lens)
        if case["inlet"]:
            L.set_x_boundaries(lbm.XBC_INLET_OUTLET, *INLET)
        L.init_device(*_fields(nx, ny, case["c2"], case["init"], gen))
        fields = torch.empty(3, ny, nx, dtype=torch.float64, device="cuda")
        frame = None if case["dtype"] == "f64" else torch.empty(3, ny, nx, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        return {"kind": "frame", "lattice": L, "steps": case["steps"], "lens": lens, "fields": fields, "frame": frame}
    if case["kind"] == "pool":
        specs = _pool_specs(case)
        P = lbm.Pool(sum(lbm.Pool.slot_bytes(s["nx"], s["ny"], case["dtype"]) for s in specs), case["dtype"])
        P.set_mode({"grouped": lbm.GROUPED, "graph": lbm.GRAPH, "persistent": lbm.PERSISTENT}[case["mode"]])
        slots = []
        for s in specs:
            f = _fields(s["nx"], s["ny"], s["c2"], "pulse", gen)
            torch.cuda.synchronize()
            slots.append(P.add(s["nx"], s["ny"], s["tau"], s["c2"]))
            P.init_device(slots[-1], *f)
            P.sync()
        steps = np.array([s["steps"] for s in specs], dtype=np.int32)
        done = [(k, None if case["dtype"] == "f64" else torch.empty(3, s["ny"], s["nx"], dtype=torch.float32))
                for k, s in zip(slots, specs) if s["done"]]
        return {"kind": "pool", "pool": P, "slots": slots, "steps": steps, "done": done}
    nx, ny = case["nx"], case["ny"]
    L = lbm.Lattice(nx, ny, case["tau"], case["c2"], case["dtype"])
    host = [t.cpu().numpy() for t in _fields(nx, ny, case["c2"], case["init"], gen)]
    return {"kind": "job", "lattice": L, "steps": case["steps"], "host": host}


def run(state):
    if state["kind"] == "frame":
        L, fields = state["lattice"], state["fields"]
        if state["lens"] is not None:
            L.set_c2_field_device(state["lens"])
        L.step(state["steps"])
        totals = L.moments_device(fields[0], fields[1], fields[2])
        if state["frame"] is None:
            return {"fields": fields, "totals": totals}
        state["frame"].copy_(fields)
        return {"fields": state["frame"]}
    if state["kind"] == "pool":
        P = state["pool"]
        P.step(state["slots"], state["steps"])
        out = []
        for slot, frame in state["done"]:
            rho, ux, uy, _, _ = P.moments(slot)
            if frame is None:
                out.append((rho, ux, uy))
            else:
                for k, a in enumerate((rho, ux, uy)):
                    frame[k].copy_(torch.from_numpy(a))
                out.append(frame)
        return out
    L = state["lattice"]
    L.init(*state["host"])
    L.step(state["steps"])
    return L.get_f()


# ---------------------------------------------------------------------------
# What a pass cannot do without


def work(case):
    es = ESIZE[case["dtype"]]
    if case["kind"] == "frame":
        n = case["nx"] * case["ny"]
        extra = (8 if case["field"] else 0) + 3 * (8 if case["dtype"] == "f64" else 4)
        return {"bytes": n * (18 * es + extra), "flops": FLOPS * n * case["steps"]}
    if case["kind"] == "pool":
        specs = _pool_specs(case)
        out = 8 if case["dtype"] == "f64" else 4
        return {"bytes": sum(s["nx"] * s["ny"] * (18 * es + (3 * out if s["done"] else 0)) for s in specs),
                "flops": sum(FLOPS * s["nx"] * s["ny"] * s["steps"] for s in specs)}
    n = case["nx"] * case["ny"]
    return {"bytes": n * (3 * 8 + 9 * 8), "flops": FLOPS * n * case["steps"]}


# ---------------------------------------------------------------------------
# The same in plain torch, 64 bits

_EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
_EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
_W = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


def _evolve(rho, ux, uy, tau, c2, steps, model="forcing", inlet=None):
    """Populations after `steps` steps from equilibrium; c2 a number or a field."""
    dev = rho.device
    ny, nx = rho.shape
    e = torch.tensor([_EX, _EY], dtype=torch.float64, device=dev)
    w = torch.tensor(_W, dtype=torch.float64, device=dev)[:, None, None]
    eq = model == "equilibrium"
    first = torch.ones(9, 1, 1, dtype=torch.float64, device=dev)
    if eq:  # moving populations carry 3 c^2 in place of 1, the rest population takes the balance
        first[1:] = 3 * c2
        first[0] = 9 / 4 - 15 / 4 * c2

    def equilibrium(r, u):
        eu = (e.t() @ u.reshape(2, -1)).reshape(9, *r.shape)
        return w * r * (first + 3 * eu + 4.5 * eu * eu - 1.5 * (u * u).sum(0))

    f = equilibrium(rho, torch.stack([ux, uy]))
    for t in range(steps):
        r = f.sum(0)
        u = (e @ f.reshape(9, -1)).reshape(2, ny, nx) / r
        post = f + (equilibrium(r, u) - f) / tau
        if not eq:
            g = torch.stack([(torch.roll(r, -1, 1) - torch.roll(r, 1, 1)) / 2,
                             (torch.roll(r, -1, 0) - torch.roll(r, 1, 0)) / 2]) * (1 / 3 - c2)
            post += 3 * w * (e.t() @ g.reshape(2, -1)).reshape(9, ny, nx)
        if inlet is not None:  # the end columns emit rest equilibria; what crosses the seam is that of the column it enters
            rin = 1.0 + inlet[0] * math.sin(2 * math.pi * t / inlet[1])
            rest = (w * first)[:, :, 0]
            for i in range(9):
                post[i, :, 0] = rest[i] * (1.0 if _EX[i] < 0 else rin)
                post[i, :, -1] = rest[i] * (rin if _EX[i] > 0 else 1.0)
        f = torch.stack([torch.roll(post[i], (_EY[i], _EX[i]), (0, 1)) for i in range(9)])
    return f


def _moments(f):
    e = torch.tensor([_EX, _EY], dtype=torch.float64, device=f.device)
    r = f.sum(0)
    j = (e @ f.reshape(9, -1)).reshape(2, *r.shape)
    return torch.stack([r, j[0] / r, j[1] / r]), torch.stack([r.sum(), j[0].sum(), j[1].sum()])


MOST_EXACT = 1_500_000_000  # site updates of the plain form that take some seconds


def exact(case, seed):
    gen = _gen(seed)
    if case["kind"] == "pool":
        out, left = [], MOST_EXACT
        for s in _pool_specs(case):
            f = _fields(s["nx"], s["ny"], s["c2"], "pulse", gen)
            if not s["done"]:
                continue
            cost = max(s["nx"] * s["ny"], 50_000) * s["steps"]
            if cost > left:
                out.append((None, None, None) if case["dtype"] == "f64" else None)
                continue
            left -= cost
            m = _moments(_evolve(*f, s["tau"], s["c2"], s["steps"]))[0]
            out.append((m[0], m[1], m[2]) if case["dtype"] == "f64" else m)
        return out
    nx, ny = case["nx"], case["ny"]
    if max(nx * ny, 50_000) * case["steps"] > MOST_EXACT:
        return None
    f = _fields(nx, ny, case["c2"], case["init"], gen)
    if case["kind"] == "job":
        return _evolve(*f, case["tau"], case["c2"], case["steps"])
    c2 = _lens(nx, ny, case["c2"]) if case["field"] else case["c2"]
    f = _evolve(*f, case["tau"], c2, case["steps"], case["model"], INLET if case["inlet"] else None)
    fields, totals = _moments(f)
    return {"fields": fields, "totals": totals} if case["dtype"] == "f64" else {"fields": fields}
