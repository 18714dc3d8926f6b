"""Cases that stand for the work a program gives to this library, and how one
pass of each is run: plans made once, then objectives, gradients, adjoints,
Hessian-vector products and autograd steps through the public entry points.

A case is a dict of plain values.  ``kind`` names the objective:

* ``mesh``    -- MeshObjective on a structured hex mesh, a chain, a ring of
                 k-node elements or uniformly random connectivity;
* ``dense``   -- DenseObjective, the row reduction;
* ``bdense``  -- BatchedDense, the products on the matrix cores;
* ``batch``   -- MeshBatch, uneven hex meshes in one launch;
* ``paper``   -- Laplace1D, ||A(3x) - b||^2 with gradients in x and b;
* ``program`` -- a composed Program (every construct, segments, or the
                 element objective).

``op`` is what a pass does: ``gradient`` (f and the gradient in one call),
``adjoint`` (the objective, then its adjoint with a device seed), ``hvp`` (a
Hessian-vector and a Jacobian-vector product) or ``step`` (forward and
backward through torch.autograd, as a training step does).  Inputs are drawn
on the device from the seed, with the distributions of the seeded workloads
in ``paper_2507_13204_amd.inputs``.
"""
from __future__ import annotations

import math

import torch

from paper_2507_13204_amd import inputs, pgrad

DTYPES = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # The 1D chain at the largest size of the paper's sweep: a call that is
        # all latency, as inside an optimiser on a small model.
        {"name": "chain_10k", "kind": "mesh", "conn": "chain", "n": 10_000, "k": 2,
         "dtype": "f64", "adjoint": "atomic", "op": "gradient"},
        # The paper's own example, gradients in both of its operands.
        {"name": "paper_10k", "kind": "paper", "n": 10_000, "dtype": "f64", "op": "gradient"},
        # The headline workload: one gradient of the 128^3 hex mesh.
        {"name": "hex128_f64", "kind": "mesh", "conn": "hex", "n": 128, "k": 8,
         "dtype": "f64", "adjoint": "atomic", "op": "gradient"},
        # A training step in FP32 storage on a mesh of an odd, middling size.
        {"name": "hex61_f32_step", "kind": "mesh", "conn": "hex", "n": 61, "k": 8,
         "dtype": "f32", "adjoint": "atomic", "op": "step"},
        # A bitwise repeatable gradient, as a regression run or a line search
        # that compares runs asks for.
        {"name": "hex48_tiled", "kind": "mesh", "conn": "hex", "n": 48, "k": 8,
         "dtype": "f64", "adjoint": "tiled", "op": "gradient"},
        # Elements of a row length that is no power of two (a wedge or an
        # arbitrary stencil), a size that fills no whole workgroup.
        {"name": "ring_k5", "kind": "mesh", "conn": "ring", "n": 300_007, "k": 5,
         "dtype": "f64", "adjoint": "atomic", "op": "gradient"},
        # The dense row reduction at its benchmark size.
        {"name": "dense_10k", "kind": "dense", "rows": 10_000, "cols": 10_000,
         "dtype": "f64", "op": "gradient"},
        # Many samples of few features, an odd number of them; the objective
        # and its adjoint called apart, as a caller with its own tape does.
        {"name": "dense_tall_301", "kind": "dense", "rows": 50_003, "cols": 301,
         "dtype": "f64", "op": "adjoint"},
        # The batched products on the FP64 matrix cores at their benchmark size.
        {"name": "bdense_f64", "kind": "bdense", "m": 4096, "n": 1024,
         "dtype": "f64", "op": "gradient"},
        # A training step of the FP32 products at a size that fills no whole
        # tiles.
        {"name": "bdense_f32_step", "kind": "bdense", "m": 3000, "n": 500,
         "dtype": "f32", "op": "step"},
        # 256 uneven hex meshes, sides log-uniform in [10, 100], in one call.
        {"name": "batch_256", "kind": "batch", "n_inst": 256, "lo": 10, "hi": 100,
         "dtype": "f64", "op": "gradient"},
        # A composed program that uses every construct: stencil, scan, gather,
        # products and maps, with active and inactive branches.
        {"name": "program_mix", "kind": "program", "form": "mix", "n": 300_007,
         "n_elems": 200_003, "k": 8, "op": "gradient"},
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], uniform in its logarithm, odd half the time."""
    v = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["mesh", "mesh", "mesh", "mesh", "dense", "dense", "bdense", "bdense",
                       "batch", "paper", "program", "program"])
    if kind == "mesh":
        conn = rng.choice(["hex", "hex", "chain", "ring", "random"])
        k = {"hex": 8, "chain": 2}.get(conn) or rng.choice([2, 3, 4, 5, 6, 8, 10])
        n = {"hex": lambda: _log(rng, 6, 128), "chain": lambda: _log(rng, 100, 1_000_000),
             "ring": lambda: _log(rng, 1_000, 1_000_000),
             "random": lambda: _log(rng, 1_000, 300_000)}[conn]()
        adjoint = rng.choice(["atomic", "atomic", "atomic", "gather", "tiled", "colour"])
        if adjoint != "atomic":  # these build their tables on the host: middling sizes
            n = min(n, {"hex": 64}.get(conn, 100_000))
            if conn == "random" and adjoint == "colour":
                adjoint = "gather"  # a random node can need more colours than there are
        op = rng.choice(["gradient", "gradient", "adjoint", "hvp", "step"])
        return {"kind": kind, "conn": conn, "n": n, "k": k, "dtype": rng.choice(["f64", "f64", "f32"]),
                "adjoint": adjoint, "op": op}
    if kind == "dense":
        cols = _log(rng, 16, 20_001)
        rows = _log(rng, 16, min(100_000, 80_000_000 // cols))
        return {"kind": kind, "rows": rows, "cols": cols, "dtype": rng.choice(["f64", "f64", "f32"]),
                "op": rng.choice(["gradient", "adjoint", "step"])}
    if kind == "bdense":
        return {"kind": kind, "m": _log(rng, 100, 4096), "n": _log(rng, 16, 1024),
                "dtype": rng.choice(["f64", "f32"]), "op": rng.choice(["gradient", "adjoint", "step"])}
    if kind == "batch":
        return {"kind": kind, "n_inst": _log(rng, 4, 128), "lo": 10, "hi": rng.choice([20, 50, 100]),
                "dtype": rng.choice(["f64", "f64", "f32"]), "op": rng.choice(["gradient", "step"])}
    if kind == "paper":
        return {"kind": kind, "n": _log(rng, 10, 3_000_000), "dtype": rng.choice(["f64", "f32"]),
                "op": "gradient"}
    form = rng.choice(["mix", "segments", "mesh"])
    n = _log(rng, 6, 96) if form == "mesh" else _log(rng, 1_000, 1_000_000)
    return {"kind": kind, "form": form, "n": n,
            "n_elems": (n - 1) ** 3 if form == "mesh" else _log(rng, 1_000, 500_000),
            "k": 8 if form == "mesh" else rng.choice([3, 4, 5, 8]),
            "op": rng.choice(["gradient", "gradient", "step"])}


# ------------------------------------------------------------------- inputs

class _Draws:
    """Device tensors drawn from one seed in a fixed order."""

    def __init__(self, seed, dtype=torch.float64):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))
        self.dtype = dtype

    def uniform(self, shape, lo, hi):
        t = torch.rand(shape, dtype=torch.float64, device="cuda", generator=self.gen)
        return t.mul_(hi - lo).add_(lo).to(self.dtype)

    def normal(self, shape, scale=1.0):
        t = torch.randn(shape, dtype=torch.float64, device="cuda", generator=self.gen)
        return t.mul_(scale).to(self.dtype)

    def index(self, shape, top):
        return torch.randint(0, top, shape, dtype=torch.int32, device="cuda", generator=self.gen)


def _hex_conn(s):
    """Lexicographic connectivity of an s^3-node hex mesh (see inputs.hex_conn)."""
    i = torch.arange(s - 1, device="cuda")
    base = (i[None, None, :] + s * (i[None, :, None] + s * i[:, None, None])).reshape(-1, 1)
    corner = torch.tensor([(c & 1) + s * ((c >> 1 & 1) + s * (c >> 2)) for c in range(8)],
                          device="cuda")
    return (base + corner).to(torch.int32)


def _mesh_sizes(case):
    """(nodes, elements) of a mesh case."""
    n = case["n"]
    if case["conn"] == "hex":
        return n ** 3, (n - 1) ** 3
    if case["conn"] == "chain":
        return n, n - 1
    if case["conn"] == "ring":
        return n, n
    return n, 2 * n  # random: two elements per node


def _mesh_inputs(case, seed):
    d = _Draws(seed, DTYPES[case["dtype"]])
    N, E = _mesh_sizes(case)
    k, conn = case["k"], case["conn"]
    x = d.uniform((N,), -1.0, 1.0)
    if conn == "chain":
        e = torch.arange(E, device="cuda")
        c = torch.stack([e, e + 1], 1).to(torch.int32)
        # the element gradient of a unit interval cut into n cells
        B = torch.tensor([[-float(N), float(N)]], dtype=d.dtype, device="cuda").repeat(E, 1)
        w = torch.full((E,), 1.0 / N, dtype=d.dtype, device="cuda")
    else:
        if conn == "hex":
            c = _hex_conn(case["n"])
        elif conn == "ring":
            c = (torch.arange(E, device="cuda")[:, None] + torch.arange(k, device="cuda")) % N
            c = c.to(torch.int32)
        else:
            c = d.index((E, k), N)
        B = d.normal((E, k))
        w = d.uniform((E,), 0.5, 1.5)
    v = d.uniform((N,), -1.0, 1.0)
    return c.contiguous(), B, w, x, v


def _batch_inputs(case, seed):
    d = _Draws(seed, DTYPES[case["dtype"]])
    sides, _ = inputs.uneven_sides(case["n_inst"], lo=case["lo"], hi=case["hi"])
    inst, conns, no, eo = [], [], 0, 0
    for s in (int(s) for s in sides):
        inst.append((s ** 3, (s - 1) ** 3, no, eo))
        conns.append(_hex_conn(s))
        no += s ** 3
        eo += (s - 1) ** 3
    return inst, torch.cat(conns), d.normal((eo, 8)), d.uniform((eo,), 0.5, 1.5), \
        d.uniform((no,), -1.0, 1.0)


def _dense_inputs(case, seed):
    d = _Draws(seed, DTYPES[case["dtype"]])
    rows, cols = case["rows"], case["cols"]
    return d.normal((rows, cols), 1.0 / math.sqrt(cols)), d.uniform((rows,), 0.5, 1.5), \
        d.uniform((cols,), -1.0, 1.0)


def _bdense_inputs(case, seed):
    d = _Draws(seed, DTYPES[case["dtype"]])
    m, n = case["m"], case["n"]
    return d.normal((m, m), 1.0 / math.sqrt(m)), d.uniform((m, n), 0.5, 1.5), \
        d.uniform((m, n), -1.0, 1.0)


def _program_inputs(case, seed):
    """The construct list (array operands on the device) and the input vectors."""
    d = _Draws(seed)
    form, n, E, k = case["form"], case["n"], case["n_elems"], case["k"]
    if form == "mesh":
        x = d.uniform((n ** 3,), -1.0, 1.0)
        spec = [("input", n ** 3), ("gather", 0, _hex_conn(n), d.normal((E, 8))), ("map", 1, "psi"),
                ("const", d.uniform((E,), 0.5, 1.5)), ("mul", 2, 3), ("sum", 4)]
        return spec, [x]
    if form == "segments":
        off = inputs.segment_offsets(max(3, n // 20), 20.0, seed=6)
        n = int(off[-1])
        offs = torch.from_numpy(off).to("cuda")
        x, c = d.uniform((n,), -1.0, 1.0), d.uniform((n,), -1.0, 1.0)
        spec = [("input", n), ("segsum", 0, offs), ("map", 1, "psi"), ("bcast", 2, offs),
                ("mul", 3, 0), ("const", c), ("mul", 0, 5), ("segsum", 6, offs),
                ("scale", 7, 0.5), ("bcast", 8, offs), ("add", 4, 1.0, 9, 1.0), ("sum", 10)]
        return spec, [x]
    x, y, c = (d.uniform((n,), -1.0, 1.0) for _ in range(3))
    coef = [0.31, -0.52, 0.44, 0.17, -0.29]
    conn, B, w = d.index((E, k), n), d.normal((E, k), 1.0 / math.sqrt(k)), d.uniform((E,), 0.5, 1.5)
    spec = [("input", n), ("input", n), ("const", c), ("stencil", 0, [-2, -1, 0, 1, 3], coef),
            ("scale", 1, -0.7), ("mul", 3, 4), ("add", 5, 0.3, 2, 1.1), ("map", 6, "psi"),
            ("scan", 7), ("scale", 8, 1.0 / n), ("stencil", 2, [0, 1], [1.0, -1.0]),
            ("add", 9, 1.0, 10, 0.5), ("gather", 11, conn, B), ("mul", 12, 12),
            ("map", 12, "square"), ("add", 13, 0.25, 14, 0.75), ("const", w), ("mul", 15, 16),
            ("sum", 17)]
    return spec, [x, y]


# ------------------------------------------------------------ the measured path

def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "mesh":
        conn, B, w, x, v = _mesh_inputs(case, seed)
        N, _ = _mesh_sizes(case)
        st["obj"] = pgrad.MeshObjective(conn, B, w, N, adjoint=case["adjoint"])
        st["fn"] = pgrad.MeshFn
        st["v"] = v
    elif kind == "dense":
        A, w, x = _dense_inputs(case, seed)
        st["obj"] = pgrad.DenseObjective(A, w)
        st["fn"] = pgrad.DenseFn
    elif kind == "bdense":
        A, W, x = _bdense_inputs(case, seed)
        st["obj"] = pgrad.BatchedDense(A, W)
        st["fn"] = pgrad.BatchedDenseFn
    elif kind == "batch":
        inst, conn, B, w, x = _batch_inputs(case, seed)
        st["obj"] = pgrad.MeshBatch(inst, conn, B, w)
        st["fn"] = pgrad.MeshBatchFn
        st["seed"] = torch.ones(len(inst), dtype=torch.float64, device="cuda")
    elif kind == "paper":
        d = _Draws(seed, DTYPES[case["dtype"]])
        x, st["b"] = (d.uniform((case["n"],), -1.0, 1.0) for _ in range(2))
        st["obj"] = pgrad.Laplace1D(case["n"], dtype=d.dtype)
    else:
        spec, xs = _program_inputs(case, seed)
        st["prog"] = pgrad.Program.from_spec(spec, device="cuda").plan("cuda")
        st["xs"] = [t.requires_grad_(case["op"] == "step") for t in xs]
        return st
    if case["op"] == "adjoint":
        st["fbar"] = torch.full((1,), 0.75, dtype=torch.float64, device="cuda")
    st["x"] = x.requires_grad_(case["op"] == "step")
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if case["kind"] == "program":
        if op == "gradient":
            f, grads = st["prog"].run(st["xs"])
            return [f, *grads]
        for x in st["xs"]:
            x.grad = None
        f = pgrad.ProgramFn.apply(st["prog"], *st["xs"])
        f.backward()
        return [f.detach(), *(x.grad for x in st["xs"])]
    obj, x = st["obj"], st["x"]
    if case["kind"] == "paper":
        return list(obj.gradient(x, st["b"]))
    if op == "gradient":
        return list(obj.gradient(x))
    if op == "adjoint":
        return [obj.objective(x), obj.adjoint(x, st["fbar"])]
    if op == "hvp":
        return [obj.jvp(x, st["v"]), obj.hvp(x, st["v"])]
    x.grad = None
    f = st["fn"].apply(x, obj)
    f.backward(st.get("seed"))
    return [f.detach(), x.grad]


# --------------------------------------------------- what a pass cannot do without

def work(case):
    es = 4 if case.get("dtype") == "f32" else 8
    kind, op = case["kind"], case["op"]
    if kind == "mesh":
        N, E = _mesh_sizes(case)
        k = case["k"]
        # rows (conn, B, w) and x read once, one vector written; the HVP and
        # the JVP are two results that share the rows and the direction
        nbytes = E * (4 * k + es * k + es) + es * N * (3 if op == "hvp" else 2)
        return {"bytes": nbytes, "flops": E * (4 * k + 20)}
    if kind == "batch":
        sides, _ = inputs.uneven_sides(case["n_inst"], lo=case["lo"], hi=case["hi"])
        E, N = int(((sides - 1) ** 3).sum()), int((sides ** 3).sum())
        return {"bytes": E * (32 + 9 * es) + 2 * es * N, "flops": E * 52}
    if kind == "dense":
        r, c = case["rows"], case["cols"]
        return {"bytes": es * (r * c + r + 2 * c), "flops": 4 * r * c}
    if kind == "bdense":
        m, n = case["m"], case["n"]
        return {"bytes": es * (m * m + 3 * m * n), "flops": 4 * m * m * n}
    if kind == "paper":
        return {"bytes": 4 * es * case["n"], "flops": 20 * case["n"]}
    n, E, k = case["n"], case["n_elems"], case["k"]
    if case["form"] == "mesh":
        return {"bytes": E * (32 + 72) + 16 * n ** 3, "flops": E * 52}
    if case["form"] == "segments":
        return {"bytes": 8 * (3 * n + n // 20), "flops": 12 * n}
    # inputs, the constants and the gather's rows read once, two gradients written
    return {"bytes": 8 * 5 * n + E * (12 * k + 8), "flops": 60 * n + E * (4 * k + 10)}


# ------------------------------------------------------- the same in plain torch

def _psi(s):
    return 0.5 * s * s + 0.5 * torch.log1p(s * s)


def _dpsi(s):
    return s + s / (1.0 + s * s)


def _ddpsi(s):
    q = 1.0 + s * s
    return 1.0 + (1.0 - s * s) / (q * q)


def _mesh_u(conn, B, x):
    """u_e = sum_j B[e, j] x[conn[e, j]], one column at a time."""
    u = torch.zeros(conn.shape[0], dtype=torch.float64, device="cuda")
    for j in range(conn.shape[1]):
        u += B[:, j].double() * x[conn[:, j].long()]
    return u


def _mesh_scatter(conn, B, v, n):
    g = torch.zeros(n, dtype=torch.float64, device="cuda")
    for j in range(conn.shape[1]):
        g.index_add_(0, conn[:, j].long(), v * B[:, j].double())
    return g


def _exact_program(case, seed):
    spec, xs = _program_inputs(case, seed)
    xs = [x.requires_grad_(True) for x in xs]
    views, given = [], list(xs)
    for o in spec:
        k = o[0]
        a = views[o[1]] if k not in ("input", "const") else None
        if k == "input":
            views.append(given.pop(0))
        elif k == "const":
            views.append(o[1])
        elif k == "scale":
            views.append(o[2] * a)
        elif k == "stencil":
            n = a.numel()
            y = torch.zeros_like(a)
            for off, c in zip(o[2], o[3]):
                lo, hi = max(0, -off), min(n, n - off)
                y = y + torch.nn.functional.pad(c * a[lo + off:hi + off], (lo, n - hi))
            views.append(y)
        elif k == "gather":
            views.append(sum(o[3][:, j] * a[o[2][:, j].long()] for j in range(o[2].shape[1])))
        elif k == "add":
            views.append(o[2] * a + o[4] * views[o[3]])
        elif k == "mul":
            views.append(a * views[o[2]])
        elif k == "map":
            views.append(_psi(a) if o[2] == "psi" else a * a)
        elif k == "scan":
            views.append(torch.cumsum(a, 0))
        elif k == "segsum":
            seg = torch.repeat_interleave(torch.diff(o[2]))
            y = torch.zeros(o[2].numel() - 1, dtype=torch.float64, device="cuda")
            views.append(y.index_add(0, seg, a))
        elif k == "bcast":
            views.append(a[torch.repeat_interleave(torch.diff(o[2]))])
        else:
            views.append(a.sum())
    return [views[-1].detach(), *torch.autograd.grad(views[-1], xs)]


def exact(case, seed):
    kind, op = case["kind"], case["op"]
    fb = 0.75 if op == "adjoint" else 1.0
    if kind == "program":
        return _exact_program(case, seed)
    if kind == "mesh":
        conn, B, w, x, v = _mesh_inputs(case, seed)
        x, w, v = x.double(), w.double(), v.double()
        u = _mesh_u(conn, B, x)
        if op == "hvp":
            q = _mesh_u(conn, B, v)
            return [(w * _dpsi(u) * q).sum(), _mesh_scatter(conn, B, w * _ddpsi(u) * q, x.numel())]
        return [(w * _psi(u)).sum(), _mesh_scatter(conn, B, fb * w * _dpsi(u), x.numel())]
    if kind == "batch":
        inst, conn, B, w, x = _batch_inputs(case, seed)
        f, g = [], []
        for nn, ne, no, eo in inst:
            c, b, we, xe = conn[eo:eo + ne], B[eo:eo + ne], w[eo:eo + ne].double(), x[no:no + nn].double()
            u = _mesh_u(c, b, xe)
            f.append((we * _psi(u)).sum())
            g.append(_mesh_scatter(c, b, we * _dpsi(u), nn))
        return [torch.stack(f), torch.cat(g)]
    if kind == "dense":
        A, w, x = (t.double() for t in _dense_inputs(case, seed))
        r = A @ x
        return [(w * _psi(r)).sum(), fb * (A.t() @ (w * _dpsi(r)))]
    if kind == "bdense":
        A, W, X = (t.double() for t in _bdense_inputs(case, seed))
        Y = A @ X
        return [(W * _psi(Y)).sum(), fb * (A.t() @ (W * _dpsi(Y)))]
    d = _Draws(seed, DTYPES[case["dtype"]])
    x, b = (d.uniform((case["n"],), -1.0, 1.0).double() for _ in range(2))

    def lap(t):
        z = torch.nn.functional.pad(t, (1, 1))
        return 2.0 * t - z[:-2] - z[2:]

    r = lap(3.0 * x) - b
    return [(r * r).sum(), 6.0 * lap(r), -2.0 * r]
