"""The work that a user of this framework has it do, as cases to be timed.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (grids on the GPU, the plan / batch / server), `run` is one pass
through the public entry points, `work` what such a pass cannot do without and
`exact` its result in 64 bits.  A program that steps a grid in time goes on
from where the last call ended, and so do the passes here.
"""
import math
import random

import numpy as np
import torch

from paper_2310_16298_amd import stencil as st

SHAPES = {"star": st.STAR, "box": st.BOX, "general": st.GENERAL}
BCS = {"zero": st.BC_ZERO, "periodic": st.BC_PERIODIC}
DTYPES = {"f32": st.F32, "f64": st.F64}
PATHS = {"auto": st.PATH_AUTO, "bf16x3": st.PATH_MFMA_BF16X3, "f16x3": st.PATH_MFMA_F16X3}
TORCH = {"f32": torch.float32, "f64": torch.float64}
DEVICE = "cuda"


def listed():
    return [
        # one explicit step of the smallest Table 3 grid, as a solver that owns its time loop calls it: latency
        {"name": "apply_64_f64", "kind": "apply", "d0": 64, "d1": 64, "d2": 0, "shape": "box", "radius": 1,
         "bc": "zero", "dtype": "f64"},
        # the latency configuration: 2D diffusion, 512 x 512 FP64 five-point star, 10 steps
        {"name": "star2d_512_f64", "kind": "solve", "d0": 512, "d1": 512, "d2": 0, "shape": "star", "radius": 1,
         "bc": "zero", "dtype": "f64", "path": "auto", "steps": 10},
        # the headline benchmark, two of its orders: 8192 x 8192 FP32 box, periodic, 100 steps
        {"name": "box2d_8192_f32_r2", "kind": "solve", "d0": 8192, "d1": 8192, "d2": 0, "shape": "box", "radius": 2,
         "bc": "periodic", "dtype": "f32", "path": "auto", "steps": 100},
        {"name": "box2d_8192_f32_r4", "kind": "solve", "d0": 8192, "d1": 8192, "d2": 0, "shape": "box", "radius": 4,
         "bc": "periodic", "dtype": "f32", "path": "auto", "steps": 100},
        # a domain whose extents nobody rounded: high-order star (wave equation) on 1021 x 1531
        {"name": "ragged2d_f32_r3", "kind": "solve", "d0": 1021, "d1": 1531, "d2": 0, "shape": "star", "radius": 3,
         "bc": "zero", "dtype": "f32", "path": "auto", "steps": 50},
        # the 3D benchmark grid: order-4 star (seismic stencil) at 512^3
        {"name": "star3d_512_f32_r4", "kind": "solve", "d0": 512, "d1": 512, "d2": 512, "shape": "star", "radius": 4,
         "bc": "zero", "dtype": "f32", "path": "auto", "steps": 50},
        # the arithmetic-bound end: 343-point box at 256^3
        {"name": "box3d_256_f32_r3", "kind": "solve", "d0": 256, "d1": 256, "d2": 256, "shape": "box", "radius": 3,
         "bc": "zero", "dtype": "f32", "path": "auto", "steps": 10},
        # 3D in double precision on odd extents: 27-point box
        {"name": "ragged3d_f64_r1", "kind": "solve", "d0": 203, "d1": 150, "d2": 177, "shape": "box", "radius": 1,
         "bc": "periodic", "dtype": "f64", "path": "auto", "steps": 20},
        # the mixed-precision benchmark: BF16 hi/lo operands, 4096 x 4096 box of order 2, 200 steps
        {"name": "mixed2d_4096_bf16x3", "kind": "solve", "d0": 4096, "d1": 4096, "d2": 0, "shape": "box", "radius": 2,
         "bc": "periodic", "dtype": "f32", "path": "bf16x3", "steps": 200},
        # an irregular order-4 stencil (scattered weights and a diagonal) on the benchmark grid
        {"name": "general2d_8192_f32", "kind": "solve", "d0": 8192, "d1": 8192, "d2": 0, "shape": "general",
         "radius": 4, "taps": 17, "bc": "periodic", "dtype": "f32", "path": "auto", "steps": 30},
        # a batch of the paper's Table 3 shapes, FP64, 10 steps: 64^2..512^2 and 8^3..64^3, star and box, order 1..3
        {"name": "batch_table3_f64", "kind": "batch", "mix": 7, "grids": 120, "dtype": "f64", "max2d": 512,
         "max3d": 64, "steps": 10},
        # a burst of requests of mixed sizes at the serving loop
        {"name": "serve_mix_f32", "kind": "serve", "mix": 11, "requests": 16, "max2d": 2048, "max3d": 192,
         "max_steps": 100},
    ]


# ------------------------------------------------------------------- drawing

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even_or_odd(rng, v):
    """Half of the extents are multiples of 16, as people choose them; the others are what comes."""
    return max(16, v // 16 * 16) if rng.random() < 0.5 else v


def _taps(case):
    r, nd = case["radius"], 3 if case["d2"] else 2
    if case["shape"] == "general":
        return case["taps"]
    return (2 * r + 1) ** nd if case["shape"] == "box" else 2 * r * nd + 1


def _points(case):
    return case["d0"] * case["d1"] * (case["d2"] or 1)


def _bounded(case, flops, most_steps):
    """Sizes and steps within `flops` useful operations and 3e9 point-steps."""
    cap = min(flops / (2.0 * _taps(case)), 3.0e9)
    while _points(case) > cap:
        k = max(("d0", "d1", "d2"), key=lambda d: case[d])
        case[k] = max(16, case[k] // 2 + case[k] % 2)
    if "steps" in case:
        case["steps"] = max(1, min(case["steps"], int(cap / _points(case)), most_steps))
    return case


def draw(rng):
    kind = rng.choice(["apply", "solve2d", "solve2d", "solve2d", "solve3d", "solve3d", "split", "general", "batch",
                       "serve"])
    if kind == "batch":
        return {"kind": "batch", "mix": rng.randrange(1 << 20), "grids": _log(rng, 8, 120),
                "dtype": rng.choice(["f32", "f64"]), "max2d": rng.choice([128, 256, 512]),
                "max3d": rng.choice([16, 32, 64]), "steps": _log(rng, 2, 30)}
    if kind == "serve":
        return {"kind": "serve", "mix": rng.randrange(1 << 20), "requests": _log(rng, 2, 16),
                "max2d": rng.choice([512, 1024, 2048]), "max3d": rng.choice([64, 128, 192]),
                "max_steps": _log(rng, 10, 100)}
    c = {"kind": "apply" if kind == "apply" else "solve", "d0": 0, "d1": 0, "d2": 0,
         "shape": rng.choice(["star", "box"]), "radius": rng.randint(1, 4), "bc": rng.choice(["zero", "periodic"]),
         "dtype": rng.choice(["f32", "f64"])}
    if kind != "apply":
        c["path"], c["steps"] = "auto", _log(rng, 4, 200)
    if kind in ("solve3d", "split") and (kind == "solve3d" or rng.random() < 0.4):
        for k in ("d0", "d1", "d2"):
            c[k] = _even_or_odd(rng, _log(rng, 24, 512))
    else:
        side = (48, 1024) if kind == "apply" else (48, 8192)
        for k in ("d0", "d1"):
            c[k] = _even_or_odd(rng, _log(rng, *side))
    flops = 1.0e11 if c["d2"] else 3.0e11
    if kind == "split":
        c["dtype"], c["path"] = "f32", rng.choice(["bf16x3", "f16x3"])
        flops *= 0.5
    if kind == "general":
        c["shape"], c["radius"] = "general", rng.randint(2, 4)
        c["taps"] = rng.randint(4, (2 * c["radius"] + 1) ** 2 * 2 // 3)
    return _bounded(c, flops, 200)


# -------------------------------------------------------------------- inputs

def _mask(nd, r, shape):
    w = 2 * r + 1
    if shape != "star":
        return np.ones((w,) * nd, dtype=bool)
    off = np.stack(np.meshgrid(*([np.arange(w) - r] * nd), indexing="ij"))
    return (off != 0).sum(0) <= 1


def _coefficients(nd, r, shape, seed, taps=0):
    """Positive weights that sum to 1 on the stencil's taps (FP64)."""
    rng = np.random.default_rng(seed)
    c = np.where(_mask(nd, r, shape), rng.uniform(0.05, 1.0, (2 * r + 1,) * nd), 0.0)
    if shape == "general":  # a diagonal first, then points anywhere
        keep = np.zeros(c.shape, dtype=bool)
        diag = np.arange(2 * r + 1)[:taps]
        keep[diag, diag] = True
        rest = rng.permutation(np.flatnonzero(~keep.reshape(-1)))[:taps - len(diag)]
        keep.reshape(-1)[rest] = True
        c = np.where(keep, c, 0.0)
    return c / c.sum()


def _dims(case):
    return (case["d0"], case["d1"], case["d2"]) if case["d2"] else (case["d0"], case["d1"])


def _field(dims, dtype, gen):
    """Values uniform on [-1, 1), drawn on the GPU."""
    return torch.rand(dims, dtype=TORCH[dtype], device=DEVICE, generator=gen).mul_(2).sub_(1)


def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _stencil_seed(case, seed):
    return [int(seed) & 0x7FFFFFFF, case["radius"], 3 if case["d2"] else 2]


def _batch_members(case):
    """The grids of a batch: Table 3 shapes (2D squares and 3D cubes, order 1..3)."""
    rng = random.Random(case["mix"])
    out = []
    for _ in range(case["grids"]):
        two = rng.random() < 0.6
        n = rng.choice([v for v in ((64, 128, 256, 512) if two else (8, 16, 32, 64))
                        if v <= (case["max2d"] if two else case["max3d"])])
        shape = rng.choice(["star", "box"])
        r = rng.randint(1, 3 if two or shape == "star" else 2)
        out.append({"d0": n, "d1": n, "d2": 0 if two else n, "shape": shape, "radius": r,
                    "bc": rng.choice(["zero", "periodic"])})
    return out


def _requests(case):
    """The requests of a burst: 2D squares and 3D cubes, side log-uniform, order 1..4, star or box."""
    rng = random.Random(case["mix"])
    out = []
    for _ in range(case["requests"]):
        two = rng.random() < 0.5
        n = _log(rng, 64, case["max2d"]) if two else _log(rng, 32, case["max3d"])
        c = {"d0": n, "d1": n, "d2": 0 if two else n, "shape": rng.choice(["star", "box"]),
             "radius": rng.randint(1, 4), "bc": rng.choice(["zero", "periodic"]),
             "steps": rng.randint(1, case["max_steps"])}
        out.append(_bounded(c, 1.0e10, case["max_steps"]))
    return out


def prepare(case, seed):
    gen = _gen(seed)
    if case["kind"] == "batch":
        members = _batch_members(case)
        places, total = [], 0
        for m in members:  # all grids in two pools, as a program that steps many of them keeps them
            places.append(total)
            total += (_points(m) + 63) // 64 * 64
        pools = [torch.zeros(total, dtype=TORCH[case["dtype"]], device=DEVICE) for _ in range(2)]
        plans, bufs = [], ([], [])
        for k, (m, at) in enumerate(zip(members, places)):
            for side in (0, 1):
                bufs[side].append(pools[side][at:at + _points(m)].view(_dims(m)))
            bufs[0][k].copy_(_field(_dims(m), case["dtype"], gen))
            c = _coefficients(len(_dims(m)), m["radius"], m["shape"], _stencil_seed(m, seed + k))
            plans.append(st.Plan(_dims(m), m["radius"], SHAPES[m["shape"]], c, boundary=BCS[m["bc"]],
                                 dtype=DTYPES[case["dtype"]]))
        # a program that steps an odd number of times at once goes on from the other pool
        batches = [st.Batch(plans, bufs[0], bufs[1]), st.Batch(plans, bufs[1], bufs[0])]
        return {"kind": "batch", "pools": pools, "batches": batches, "at": 0, "steps": case["steps"]}
    if case["kind"] == "serve":
        reqs = []
        for k, m in enumerate(_requests(case)):
            x = _field(_dims(m), "f32", gen)
            c = _coefficients(len(_dims(m)), m["radius"], m["shape"], _stencil_seed(m, seed + k))
            reqs.append((m, x, torch.empty_like(x), c))
        need = sum(2 * (x.numel() * 4 + 65536) + (1 << 20) for _, x, _, _ in reqs)
        return {"kind": "serve", "server": st.Server(need), "requests": reqs}
    dims = _dims(case)
    c = _coefficients(len(dims), case["radius"], case["shape"], _stencil_seed(case, seed), case.get("taps", 0))
    x = _field(dims, case["dtype"], gen)
    plan = st.Plan(dims, case["radius"], SHAPES[case["shape"]], c, boundary=BCS[case["bc"]],
                   dtype=DTYPES[case["dtype"]], path=PATHS[case.get("path", "auto")])
    return {"kind": case["kind"], "plan": plan, "x": x, "y": torch.empty_like(x), "steps": case.get("steps", 1)}


def run(state):
    if state["kind"] == "apply":
        return state["plan"].apply(state["x"], state["y"])
    if state["kind"] == "solve":
        res = state["plan"].run_steps(state["x"], state["y"], state["steps"])
        if res is not state["x"]:  # the next call goes on from this result
            state["x"], state["y"] = state["y"], state["x"]
        return res
    if state["kind"] == "batch":
        idx = state["batches"][state["at"]].run_steps(state["steps"])
        state["at"] ^= idx
        return state["pools"][state["at"]]
    server = state["server"]
    server.stream().wait_stream(torch.cuda.current_stream())  # the inputs are written
    left = set()
    for m, x, out, c in state["requests"]:
        left.add(server.submit(x, out, m["steps"], m["radius"], SHAPES[m["shape"]], c, boundary=BCS[m["bc"]]))
    busy = True
    while left:
        if busy:
            s = server.tick()
            busy = s["active"] > 0 or s["queued"] > 0
        left.difference_update(server.poll())
    return [out for _, _, out, _ in state["requests"]]


# ---------------------------------------------------------------------- work

def work(case):
    if case["kind"] == "batch":
        members = [dict(m, steps=case["steps"]) for m in _batch_members(case)]
        size = 8 if case["dtype"] == "f64" else 4
    elif case["kind"] == "serve":
        members, size = _requests(case), 4
    else:
        members, size = [case], 8 if case["dtype"] == "f64" else 4
    return {"bytes": float(sum(2 * size * _points(m) for m in members)),
            "flops": float(sum(2 * _taps(m) * _points(m) * m.get("steps", 1) for m in members))}


# --------------------------------------------------------------------- exact

def _steps64(x, c, r, bc, steps):
    """`steps` Jacobi steps of the gather coefficients c on x, in float64."""
    x = x.double()
    nd = x.dim()
    taps = [(idx, float(c[idx])) for idx in zip(*np.nonzero(c))]
    size = [n + 2 * r for n in x.shape]
    pad = torch.zeros(size, dtype=torch.float64, device=x.device)
    wrap = [torch.arange(-r, n + r, device=x.device) % n for n in x.shape]
    inner = tuple(slice(r, r + n) for n in x.shape)
    for _ in range(steps):
        if bc == "periodic":
            pad = x
            for d in range(nd):
                pad = pad.index_select(d, wrap[d])
        else:
            pad[inner] = x
        x = torch.zeros_like(x)
        for idx, w in taps:
            x.add_(pad[tuple(slice(i, i + n) for i, n in zip(idx, x.shape))], alpha=w)
    return x


def exact(case, seed):
    gen = _gen(seed)

    def one(m, x, c, steps, f32):
        if f32:
            c = c.astype(np.float32).astype(np.float64)
        return _steps64(x, c, m["radius"], m["bc"], steps)

    if case["kind"] == "batch":
        out = []
        for k, m in enumerate(_batch_members(case)):
            x = _field(_dims(m), case["dtype"], gen)
            c = _coefficients(x.dim(), m["radius"], m["shape"], _stencil_seed(m, seed + k))
            n = _points(m)
            flat = torch.zeros((n + 63) // 64 * 64, dtype=torch.float64, device=DEVICE)
            flat[:n] = one(m, x, c, case["steps"], case["dtype"] == "f32").reshape(-1)
            out.append(flat)
        return torch.cat(out)
    if case["kind"] == "serve":
        out = []
        for k, m in enumerate(_requests(case)):
            x = _field(_dims(m), "f32", gen)
            c = _coefficients(x.dim(), m["radius"], m["shape"], _stencil_seed(m, seed + k))
            out.append(one(m, x, c, m["steps"], True))
        return out
    x = _field(_dims(case), case["dtype"], gen)
    c = _coefficients(x.dim(), case["radius"], case["shape"], _stencil_seed(case, seed), case.get("taps", 0))
    return one(case, x, c, case.get("steps", 1), case["dtype"] == "f32")
