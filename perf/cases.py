"""Performance cases of the adaptive SpMV library, over the ranges it is used in.

A case is a matrix of one structural class (the classes of the library's own
sweep, its stencils and its power-law graph) with a size, a value type and
what the program does with it:

  op "spmv"    a plan is kept and y = A x is called again and again: solvers,
               graph iterations (most of the cases)
  op "levels"  every level of a multilevel hierarchy in one batch
  op "plan"    a matrix arrives, is planned with the learned selector and
               multiplied once: what a matrix that changes costs
  op "train"   one step of selector training: backward pass and Adam

Matrices are made on the GPU from integer draws and elementwise arithmetic
only, so that one seed gives the same matrix every time.
"""
import math

import torch

from paper_1210_2536_amd import spmv as G

DEV = "cuda"
TRAIN_OUT = 9         # kernel classes the selector scores
TRAIN_HID, TRAIN_IN = 64, 12


def listed():
    return [
        # latency: the 5-point Laplacian on 64 x 64 inside a small solver
        {"name": "lap5_64_f64", "op": "spmv", "kind": "grid5", "dtype": "f64", "g": 64},
        # an ordinary banded system, tuned once and kept (odd size, grid offsets)
        {"name": "band_120k_f32", "op": "spmv", "kind": "band", "dtype": "f32", "m": 120_003,
         "diags": 9, "tune": True},
        # the large structured solver: 7-point Laplacian on 256^3
        {"name": "lap7_256_f64", "op": "spmv", "kind": "grid7", "dtype": "f64", "g": 256},
        # an ordinary matrix of constant row degree and random columns
        {"name": "uniform_28k_f64", "op": "spmv", "kind": "uniform", "dtype": "f64", "m": 28_411,
         "n": 28_411, "k": 21},
        # the same structure at the top of the range, where x leaves the caches
        {"name": "uniform_730k_f32", "op": "spmv", "kind": "uniform", "dtype": "f32",
         "m": 730_117, "n": 730_117, "k": 33},
        # power-law rows, middle of the range, tuned once and kept
        {"name": "zipf_310k_f32", "op": "spmv", "kind": "zipf", "dtype": "f32", "m": 310_151,
         "alpha": 1.7, "kmin": 1, "kmax": 31_015, "tune": True},
        # power-law rows with a heavy tail, the largest matrix here
        {"name": "zipf_700k_f64", "op": "spmv", "kind": "zipf", "dtype": "f64", "m": 700_001,
         "alpha": 1.5, "kmin": 1, "kmax": 70_000},
        # a large graph: 8M vertices, exponent 2, x far beyond one L2
        {"name": "zipf_8M_f32", "op": "spmv", "kind": "zipf", "dtype": "f32", "m": 8_000_000,
         "alpha": 2.0, "kmin": 2, "kmax": 800_000},
        # dense 4x4 blocks: several unknowns per mesh node
        {"name": "blocks_400k_f64", "op": "spmv", "kind": "blocks", "dtype": "f64", "m": 400_004,
         "b": 16},
        # a multigrid cycle's residuals: 27-point stencil on 160^3 and its coarse levels
        {"name": "levels_160_f64", "op": "levels", "kind": "grid27", "dtype": "f64", "g": 160,
         "nlevels": 6},
        # a matrix that changes: plan, one product
        {"name": "plan_uniform_220k_f64", "op": "plan", "kind": "uniform", "dtype": "f64",
         "m": 220_501, "n": 220_501, "k": 24},
        # selector training at its own batch size
        {"name": "train_256", "op": "train", "batch": 256},
    ]


MOST_NNZ = 400_000_000   # no drawn case holds more entries than this


def draw(rng):
    """One more case of the same ranges."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choices(["spmv", "levels", "plan", "train"], [14, 1, 3, 1])[0]
    if op == "train":
        return {"op": op, "batch": log(64, 4096)}
    dtype = rng.choice(["f32", "f64"])
    if op == "levels":
        nl = rng.randint(3, 5)
        step = 1 << (nl - 1)
        return {"op": op, "kind": "grid27", "dtype": dtype, "nlevels": nl,
                "g": max(2, log(40, 160) // step) * step}
    kind = rng.choice(["grid5", "grid7", "band", "uniform", "uniform", "zipf", "zipf", "blocks"])
    top = 10 if op == "plan" else 1     # planning a matrix costs many products
    c = {"op": op, "kind": kind, "dtype": dtype}
    if kind == "grid5":
        c["g"] = log(32, 4096 / math.sqrt(top))
    elif kind == "grid7":
        c["g"] = log(10, 256 / top ** (1 / 3))
    elif kind == "band":
        c.update(m=log(1000, 8_000_000 / top), diags=rng.randint(3, 15))
    elif kind == "uniform":
        c.update(m=log(1000, 1_000_000 / top), k=rng.randint(8, 64))
        # rectangular now and then, as in least squares
        c["n"] = c["m"] if rng.random() < 0.75 else max(c["k"], int(c["m"] * rng.uniform(0.5, 2)))
    elif kind == "zipf":
        m = log(1000, 1_000_000 / top)
        c.update(m=m, alpha=round(rng.uniform(1.5, 2.5), 2), kmin=rng.randint(1, 2),
                 kmax=max(2, m // 10))
        if rng.random() < 0.2 and op == "spmv":
            m = log(1_000_000, 8_000_000)
            c.update(m=m, alpha=2.0, kmin=2, kmax=m // 10)
        while c["m"] * mean_degree(c) > MOST_NNZ / top:
            c["m"] = int(c["m"] * 0.9)
            c["kmax"] = c["m"] // 10
    else:
        c.update(m=log(1000, 1_000_000 / top) // 4 * 4, b=rng.randint(1, 16))
    return c


# ------------------------------------------------------------------ matrices

def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def mean_degree(case):
    """Expected row degree of a zipf case: floor of a Pareto draw on [kmin, kmax]."""
    a, lo, hi = case["alpha"] - 1.0, case["kmin"], case["kmax"]
    top = float(hi) ** -a
    norm = float(lo) ** -a - top
    # E[floor k] = sum over j >= 1 of P(k >= j)
    s, j = float(lo), lo + 1
    while j <= min(hi, 2000):
        s += (float(j) ** -a - top) / norm
        j += 1
    if hi > 2000:   # the tail as an integral
        tail = math.log(hi / 2000.0) if a == 1.0 else \
            (float(hi) ** (1 - a) - 2000.0 ** (1 - a)) / (1 - a)
        s += (tail - (hi - 2000.0) * top) / norm
    return s


def _row_ptr(length):
    rp = torch.zeros(length.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(length, 0, out=rp[1:])
    return rp


def _random_columns(gen, length, rp, n):
    """length[i] distinct ascending columns of [0, n) for each row i: sorted
    draws from [0, n - length[i]] plus their rank in the row."""
    nnz = int(rp[-1])
    rows = torch.repeat_interleave(length)
    u = torch.rand(nnz, dtype=torch.float64, device=DEV, generator=gen)
    span = (n - length + 1)[rows]
    v = torch.minimum((u * span).floor_().to(torch.int64), span - 1)
    del u, span
    key = rows.mul(1 << 32).add_(v)
    del v
    key = torch.sort(key).values
    rank = torch.arange(nnz, device=DEV) - rp[rows]
    return ((key & 0xFFFFFFFF) + rank).to(torch.int32)


def _values(gen, nnz, dtype):
    v = torch.rand(nnz, dtype=torch.float64, device=DEV, generator=gen)
    return v.mul_(2.0).sub_(1.0).to(dtype)


def _stencil(shape, offsets, coeff, dtype):
    """Stencil with Dirichlet boundaries on a row-major grid (offsets in
    ascending linear order, one coefficient each)."""
    m = math.prod(shape)
    idx = torch.arange(m, device=DEV)
    coords, rem = [], idx
    for a in range(len(shape)):
        stride = math.prod(shape[a + 1:])
        coords.append(rem // stride)
        rem = rem % stride
    strides = [math.prod(shape[a + 1:]) for a in range(len(shape))]
    inside = []
    for o in offsets:
        ok = torch.ones(m, dtype=torch.bool, device=DEV)
        for a, d in enumerate(o):
            if d:
                ok &= (coords[a] + d >= 0) & (coords[a] + d < shape[a])
        inside.append(ok)
    length = torch.zeros(m, dtype=torch.int64, device=DEV)
    for ok in inside:
        length += ok
    rp = _row_ptr(length)
    nnz = int(rp[-1])
    col = torch.empty(nnz, dtype=torch.int32, device=DEV)
    val = torch.empty(nnz, dtype=dtype, device=DEV)
    pos = rp[:-1].clone()
    for o, ok, c in zip(offsets, inside, coeff):
        p = pos[ok]
        col[p] = (idx[ok] + sum(d * s for d, s in zip(o, strides))).to(torch.int32)
        val[p] = c
        pos += ok
    return rp.to(torch.int32), col, val, m


def _band(gen, m, diags, dtype):
    """Banded rows: the diagonals 0, +-1, +-g, +-(g + 1), ... of a square grid of side g."""
    g = max(3, int(round(math.sqrt(m))))
    offs = []
    for o in (0, 1, -1, g, -g, g + 1, -(g + 1), g - 1, 1 - g, 2, -2, 2 * g, -2 * g, 2 * g + 1,
              -2 * g - 1):
        if o not in offs and -m < o < m and len(offs) < diags:
            offs.append(o)
    rp, col, val, _ = _stencil((m,), [(o,) for o in sorted(offs)], [0.0] * len(offs), dtype)
    return rp, col, _values(gen, val.numel(), dtype), m


def _blocks(gen, m, b, dtype):
    """b dense 4x4 blocks per block row."""
    mb = m // 4
    b = min(b, mb)
    length = torch.full((mb,), b, dtype=torch.int64, device=DEV)
    bcol = _random_columns(gen, length, _row_ptr(length), mb).view(mb, 1, b, 1).to(torch.int64)
    col = (bcol * 4 + torch.arange(4, device=DEV)).expand(mb, 4, b, 4)
    rp = torch.arange(m + 1, device=DEV, dtype=torch.int64) * (4 * b)
    col = col.reshape(-1).to(torch.int32)
    return rp.to(torch.int32), col, _values(gen, col.numel(), dtype), m


def matrix(case, gen):
    """(row_ptr, col, val, columns) of a case's matrix."""
    kind, dtype = case["kind"], _dtype(case)
    if kind == "grid5":
        offs = [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)]
        return _stencil((case["g"],) * 2, offs, [-1.0, -1.0, 4.0, -1.0, -1.0], dtype)
    if kind == "grid7":
        offs = [(-1, 0, 0), (0, -1, 0), (0, 0, -1), (0, 0, 0), (0, 0, 1), (0, 1, 0), (1, 0, 0)]
        return _stencil((case["g"],) * 3, offs, [-1.0] * 3 + [6.0] + [-1.0] * 3, dtype)
    if kind == "band":
        return _band(gen, case["m"], case["diags"], dtype)
    if kind == "blocks":
        return _blocks(gen, case["m"], case["b"], dtype)
    m = case["m"]
    if kind == "uniform":
        n = case["n"]
        length = torch.full((m,), case["k"], dtype=torch.int64, device=DEV)
    else:
        n = m
        a = case["alpha"] - 1.0
        lo, hi = float(case["kmin"]) ** -a, float(case["kmax"]) ** -a
        u = torch.rand(m, dtype=torch.float64, device=DEV, generator=gen)
        length = (lo - u * (lo - hi)).pow_(-1.0 / a).floor_().to(torch.int64)
        length.clamp_(case["kmin"], case["kmax"])
    rp = _row_ptr(length)
    col = _random_columns(gen, length, rp, n)
    return rp.to(torch.int32), col, _values(gen, col.numel(), dtype), n


def level_matrix(case, level):
    """Level of the 27-point hierarchy (26 / -1 on g^3) under 2x2x2 aggregation:
    27 8^l I - B x B x B with B = tridiag(1, 3 2^l - 2, 1)."""
    g = case["g"] >> level
    mid = 3.0 * 2 ** level - 2.0
    offs = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]
    coeff = [-math.prod(mid if d == 0 else 1.0 for d in o) for o in offs]
    coeff[13] += 27.0 * 8 ** level
    return _stencil((g,) * 3, offs, coeff, _dtype(case))


def _vector(gen, n, dtype):
    return _values(gen, n, dtype)


# ------------------------------------------------------------------ the contract

_MODEL = []


def _model():
    """The trained selector, loaded once as a program does."""
    if not _MODEL:
        _MODEL.append(G.default_selector())
    return _MODEL[0]


def _gen(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return gen


def _train_inputs(case, seed):
    gen = _gen(seed)
    B = case["batch"]
    shapes = [(TRAIN_HID, TRAIN_IN), (TRAIN_HID,), (TRAIN_HID, TRAIN_HID), (TRAIN_HID,),
              (TRAIN_OUT, TRAIN_HID), (TRAIN_OUT,)]
    parts = []
    for s in shapes:
        w = torch.rand(s, device=DEV, generator=gen) * 2 - 1
        parts.append((w * (math.sqrt(6.0 / s[1]) if len(s) == 2 else 0.01)).reshape(-1))
    x = torch.randn(B, TRAIN_IN, device=DEV, generator=gen)
    target = torch.rand(B, TRAIN_OUT, device=DEV, generator=gen) * math.log(20.0)
    mask = (torch.rand(B, TRAIN_OUT, device=DEV, generator=gen) < 0.7).float()
    return torch.cat(parts), x, target, mask


def prepare(case, seed):
    if case["op"] == "train":
        params, x, target, mask = _train_inputs(case, seed)
        floats = int(G.C.lib().spmv_mlp_workspace_floats(case["batch"]))
        return {"op": "train", "params": params, "x": x, "target": target, "mask": mask,
                "m": torch.zeros_like(params), "v": torch.zeros_like(params),
                "grad": torch.empty_like(params), "loss": torch.empty(1, device=DEV),
                "ws": torch.empty(floats, device=DEV), "step": 0}
    gen = _gen(seed)
    dtype = _dtype(case)
    if case["op"] == "levels":
        plans, xs, ys = [], [], []
        for level in range(case["nlevels"]):
            rp, col, val, n = level_matrix(case, level)
            plans.append(G.Plan(rp, col, val, n=n, selector="mlp", model=_model()))
            xs.append(_vector(gen, n, dtype))
            ys.append(torch.empty(n, dtype=dtype, device=DEV))
        batch = G.Batch(plans)
        batch.tune(xs, ys)
        return {"op": "levels", "batch": batch, "xs": xs, "ys": ys}
    rp, col, val, n = matrix(case, gen)
    x = _vector(gen, n, dtype)
    y = torch.empty(rp.numel() - 1, dtype=dtype, device=DEV)
    if case["op"] == "plan":
        return {"op": "plan", "csr": (rp, col, val, n), "model": _model(), "x": x, "y": y}
    plan = G.Plan(rp, col, val, n=n, selector="mlp", model=_model(),
                  autotune=bool(case.get("tune")))
    return {"op": "spmv", "plan": plan, "x": x, "y": y}


def run(state):
    op = state["op"]
    if op == "spmv":
        return state["plan"].run(state["x"], state["y"])
    if op == "levels":
        return state["batch"].run(state["xs"], state["ys"])
    if op == "plan":
        rp, col, val, n = state["csr"]
        plan = G.Plan(rp, col, val, n=n, selector="mlp", model=state["model"])
        return plan.run(state["x"], state["y"])
    state["step"] += 1
    G.mlp_backward(state["params"], state["x"], state["target"], state["mask"],
                   grad=state["grad"], ws=state["ws"], loss=state["loss"])
    G.mlp_adam(state["params"], state["grad"], state["m"], state["v"], state["step"])
    return {"grad": state["grad"], "loss": state["loss"], "params": state["params"]}


def work(case):
    if case["op"] == "train":
        B = case["batch"]
        w = TRAIN_HID * TRAIN_IN + TRAIN_HID * TRAIN_HID + TRAIN_OUT * TRAIN_HID
        # parameters and both moments read and written, gradient written, batch read
        return {"bytes": 4 * (7 * w + B * (TRAIN_IN + 2 * TRAIN_OUT)),
                "flops": 6 * B * w - 2 * B * TRAIN_HID * TRAIN_IN}
    s = 8 if case["dtype"] == "f64" else 4
    if case["op"] == "levels":
        nbytes = flops = 0
        for level in range(case["nlevels"]):
            g = case["g"] >> level
            nnz = (3 * g - 2) ** 3
            nbytes += s * nnz + 2 * s * g ** 3   # columns follow from the grid
            flops += 2 * nnz
        return {"bytes": nbytes, "flops": flops}
    kind = case["kind"]
    m = n = case["m"] if "m" in case else case["g"] ** (2 if kind == "grid5" else 3)
    if kind == "grid5":
        g = case["g"]
        nnz, index = 5 * g * g - 4 * g, 0
    elif kind == "grid7":
        g = case["g"]
        nnz, index = 7 * g ** 3 - 6 * g * g, 0
    elif kind == "band":
        nnz, index = m * case["diags"], 0        # an upper bound: the corners are cut
    elif kind == "uniform":
        n = case["n"]
        nnz = m * case["k"]
        index = 4 * nnz
    elif kind == "blocks":
        b = min(case["b"], m // 4)
        nnz = 4 * m * b
        index = nnz // 16 * 4
    else:
        nnz = int(m * mean_degree(case))
        index = 4 * nnz + 4 * (m + 1)
    if case["op"] == "plan":
        index = 4 * nnz + 4 * (m + 1)            # the CSR itself is the input
    return {"bytes": s * nnz + index + s * (n + m), "flops": 2 * nnz}


def _product(rp, col, val, x):
    """A x in float64, a row's products added in storage order (rows in
    pieces that one segment_reduce takes)."""
    rp = rp.to(torch.int64)
    x = x.double()
    ys = []
    for r0 in range(0, rp.numel() - 1, 1 << 22):
        part = rp[r0:r0 + (1 << 22) + 1]
        b, e = int(part[0]), int(part[-1])
        p = val[b:e].double() * x[col[b:e].long()]
        ys.append(torch.segment_reduce(p, "sum", offsets=part - b, initial=0.0))
    return torch.cat(ys)


def _exact_train(case, seed):
    params, x, target, mask = (t.double() for t in _train_inputs(case, seed))
    sizes = [TRAIN_HID * TRAIN_IN, TRAIN_HID, TRAIN_HID * TRAIN_HID, TRAIN_HID,
             TRAIN_OUT * TRAIN_HID, TRAIN_OUT]
    w1, b1, w2, b2, w3, b3 = torch.split(params, sizes)
    w1, w2 = w1.view(TRAIN_HID, TRAIN_IN), w2.view(TRAIN_HID, TRAIN_HID)
    w3 = w3.view(TRAIN_OUT, TRAIN_HID)
    h1 = (x @ w1.T + b1).clamp_min(0)
    h2 = (h1 @ w2.T + b2).clamp_min(0)
    r = (h2 @ w3.T + b3 - target) * mask
    count = mask.sum().clamp_min(1.0)
    ds = 2.0 * r / count
    d2 = (ds @ w3) * (h2 > 0)
    d1 = (d2 @ w2) * (h1 > 0)
    grad = torch.cat([(d1.T @ x).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0),
                      (ds.T @ h2).reshape(-1), ds.sum(0)])
    # Adam's first step: the bias corrections cancel the decay factors
    step = 1e-3 * grad / (grad.abs() + 1e-8)
    return {"grad": grad, "loss": ((r * r).sum() / count).reshape(1), "params": params - step}


def exact(case, seed):
    if case["op"] == "train":
        return _exact_train(case, seed)
    gen = _gen(seed)
    dtype = _dtype(case)
    if case["op"] == "levels":
        ys = []
        for level in range(case["nlevels"]):
            rp, col, val, n = level_matrix(case, level)
            ys.append(_product(rp, col, val, _vector(gen, n, dtype)))
        return ys
    rp, col, val, n = matrix(case, gen)
    return _product(rp, col, val, _vector(gen, n, dtype))
