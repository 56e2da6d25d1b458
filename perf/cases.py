"""The cases whose speed this framework is held to, and how one pass of each is prepared, run and checked.

Every pass calls the binding of the C ABI (``abi``) on buffers that the calling program keeps, as ``bench.py`` and
the autograd wrappers do; plans and workspaces are made once in ``prepare``.  Inputs are drawn on the GPU from the
seed alone, with the distributions of ``workloads/``.

Kinds (``draw`` spreads each over the range that its listed cases bracket):

* ``ragged`` -- row lengths to offsets, nested map (reduce) over the ragged rows, and its reverse
* ``matmul`` -- the dense nested map-map-reduce and its two products of the reverse
* ``dot``    -- fused map2 (*) + reduce (+), with its reverse for float32
* ``nbody``  -- the Euler loop around the pairwise map (reduce) with the gradient of the final kinetic energy
* ``kmeans`` -- one step (argmin + reduce-by-key), then the within-cluster SSE and its gradient
* ``batch``  -- many uneven dot / matvec expressions, forward and backward, in one launch each
* ``body``   -- a user-defined map body fused with a sum, and its generated reverse mode
* ``mriq``   -- the trigonometric reduction over samples of the Parboil shapes
"""
import math

import numpy as np
import torch

from paper_2211_00621_amd import abi, api

OPS = {"sum": abi.MX_ADD, "min": abi.MX_MIN, "max": abi.MX_MAX}
NE = {"sum": 0.0, "min": math.inf, "max": -math.inf}
DEV = "cuda"


def listed():
    return [
        # a short ragged sequence pooled by maximum, with its gradient: a few launches, bound by latency
        {"name": "ragged_max_300", "kind": "ragged", "op": "max", "rows": 300, "lmax": 500},
        # the benchmark's ragged half: 65 536 rows of log-uniform length, mean 490
        {"name": "ragged_sum_65536", "kind": "ragged", "op": "sum", "rows": 65536, "lmax": 4096},
        # the small product (a small layer, sgemm-small): one tile or two, all latency
        {"name": "matmul_small", "kind": "matmul", "m": 160, "n": 96, "k": 200},
        # the size of the paper's sgemm-medium: sides that no tile divides, too few tiles for the chip
        {"name": "matmul_medium", "kind": "matmul", "m": 1024, "n": 1056, "k": 992},
        # the benchmark's dense half
        {"name": "matmul_2048", "kind": "matmul", "m": 2048, "n": 2048, "k": 2048},
        # the benchmark's dot product with its reverse
        {"name": "dot_2e20", "kind": "dot", "dtype": "float32", "len": 1 << 20},
        # a small system: the loop's launches and latency count, not its arithmetic
        {"name": "nbody_1000", "kind": "nbody", "n": 1000, "steps": 20, "ckpt": 5},
        # the benchmark's loop, forward and checkpointed reverse
        {"name": "nbody_16384", "kind": "nbody", "n": 16384, "steps": 20, "ckpt": 5},
        # the benchmark's clustering step
        {"name": "kmeans_2e20", "kind": "kmeans", "n": 1 << 20, "d": 32, "k": 64},
        # the benchmark's batch of uneven expressions
        {"name": "batch_2048", "kind": "batch", "tasks": 2048, "smax": 1000000},
        # the benchmark's user-defined body
        {"name": "body_2e26", "kind": "body", "n": 1 << 26},
        # the benchmark's mri-q size
        {"name": "mriq_262144", "kind": "mriq", "samples": 2048, "voxels": 1 << 18},
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["ragged", "ragged", "matmul", "matmul", "dot", "nbody", "kmeans", "batch", "body", "mriq"])
    c = {"kind": kind}
    if kind == "ragged":
        c.update(op=rng.choice(["sum", "sum", "min", "max"]), rows=_log(rng, 100, 65536), lmax=_log(rng, 16, 4096))
    elif kind == "matmul":
        c.update(m=_log(rng, 48, 2048), n=_log(rng, 48, 2048), k=_log(rng, 48, 2048))
        if rng.random() < 0.5:  # half of them with sides that are multiples of 16, as layers have them
            c.update({s: -(-c[s] // 16) * 16 for s in "mnk"})
    elif kind == "dot":
        c.update(dtype=rng.choice(["float32", "float32", "int32"]), len=_log(rng, 1000, 1 << 24))
    elif kind == "nbody":
        c.update(n=_log(rng, 500, 16384), steps=20, ckpt=rng.choice([3, 5, 20]))
    elif kind == "kmeans":
        d = rng.choice([8, 16, 32, 32, 64, rng.randint(2, 64)])
        c.update(n=_log(rng, 4096, 1 << 20), d=d, k=rng.choice([10, 32, 64, rng.randint(2, 64)]))
    elif kind == "batch":
        c.update(tasks=_log(rng, 32, 2048), smax=_log(rng, 10000, 1000000))
    elif kind == "body":
        c.update(n=_log(rng, 10000, 1 << 26))
    else:
        c.update(samples=_log(rng, 128, 2048), voxels=_log(rng, 4096, 1 << 18))
    return c


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(g, lo, hi, *size):
    return torch.empty(size, dtype=torch.float32, device=DEV).uniform_(lo, hi, generator=g)


def _empty(*size, dtype=torch.float32):
    return torch.empty(size, dtype=dtype, device=DEV)


def _zeros(nbytes):
    return torch.zeros(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _ragged_inputs(c, seed):
    # lengths log-uniform in [1, lmax], one row in a hundred empty; the seed deals them out
    u = np.random.default_rng(c["rows"]).uniform(0.0, math.log(c["lmax"] + 1), c["rows"])
    lengths = np.clip(np.floor(np.exp(u)).astype(np.int64), 1, c["lmax"])
    lengths[::100] = 0
    np.random.default_rng(seed).shuffle(lengths)
    g = _gen(seed)
    total = int(lengths.sum())
    return (torch.from_numpy(lengths).to(DEV), _uniform(g, -1, 1, total), _uniform(g, -1, 1, c["rows"]))


def _matmul_inputs(c, seed):
    g = _gen(seed)
    return (_uniform(g, -1, 1, c["m"], c["k"]), _uniform(g, -1, 1, c["k"], c["n"]), _uniform(g, -1, 1, c["m"], c["n"]))


def _dot_inputs(c, seed):
    g = _gen(seed)
    if c["dtype"] == "int32":
        return tuple(torch.randint(-1000, 1001, (c["len"],), dtype=torch.int32, device=DEV, generator=g)
                     for _ in range(2))
    return _uniform(g, -1, 1, c["len"]), _uniform(g, -1, 1, c["len"]), _uniform(g, 0.5, 1.5, 1)


# Softening of about the mean spacing of the bodies.  With the 1e-3 of the benchmark the loop is chaotic at these
# sizes (tests/test_nbody_host.py): one ulp of the input moves the gradient by tens of percent, so that no result of
# it can be compared with another's.  The arithmetic is the same.
EPS2, G, DT = 0.05 ** 2, 1.0, 1e-4


def _nbody_inputs(c, seed):
    g = _gen(seed)
    pos4 = _uniform(g, 0, 1, c["n"], 4)
    pos4[:, 3] += 0.5  # masses uniform in [0.5, 1.5]
    return pos4, torch.zeros_like(pos4)


def _kmeans_inputs(c, seed):
    g = _gen(seed)
    centres = _uniform(g, -10, 10, c["k"], c["d"])
    blob = torch.randint(0, c["k"], (c["n"],), device=DEV, generator=g)
    X = torch.empty(c["n"], c["d"], device=DEV).normal_(0, 1, generator=g)
    X += centres[blob]
    return X, X[:c["k"]].clone(), _uniform(g, 0.5, 1.5, 1)


def _batch_table(c, seed):
    """Even task: dot of s elements; odd: matvec of floor(sqrt s) rows; operands on 16-byte boundaries.  The sizes are
    log-uniform; the seed deals them out to the tasks of each kind."""
    t = c["tasks"]
    s = np.exp(np.random.default_rng(t).uniform(math.log(100), math.log(c["smax"]), t)).astype(np.int64)
    order = np.random.default_rng(seed)
    s[0::2], s[1::2] = order.permutation(s[0::2]), order.permutation(s[1::2])
    kind = np.arange(t, dtype=np.int64) % 2
    rows = np.where(kind == 1, np.floor(np.sqrt(s)).astype(np.int64), 1)
    cols = -(-s // rows)
    a, b = -(-rows * cols // 4) * 4, -(-cols // 4) * 4
    a_off, b_off, o_off = (np.cumsum(x) - x for x in (a, b, rows))
    return np.stack([kind, rows, cols, a_off, b_off, o_off], axis=1), int(a.sum()), int(b.sum()), int(rows.sum())


def _batch_inputs(c, seed):
    table, na, nb, no = _batch_table(c, seed)
    g = _gen(seed)
    return table, _uniform(g, -1, 1, na), _uniform(g, -1, 1, nb), _uniform(g, -1, 1, no)


def _body_inputs(c, seed):
    g = _gen(seed)
    return _uniform(g, -1, 1, c["n"]), _uniform(g, -1, 1, c["n"]), _uniform(g, 0.5, 1.5, 1)


def _mriq_inputs(c, seed):
    g = _gen(seed)
    k = [_uniform(g, -16, 16, c["samples"]) for _ in range(3)]
    x = [_uniform(g, -0.5, 0.5, c["voxels"]) for _ in range(3)]
    return k, _uniform(g, 0, 1, c["samples"]), x


# ---------------------------------------------------------------- prepare / run
def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind, "c": c}
    if kind == "ragged":
        lengths, values, gout = _ragged_inputs(c, seed)
        s.update(lengths=lengths, values=values, gout=gout, op=OPS[c["op"]], ne=NE[c["op"]],
                 off=_empty(c["rows"] + 1, dtype=torch.int64), out=_empty(c["rows"]), gval=torch.empty_like(values),
                 ws_scan=_zeros(abi.mx_workspace_bytes(abi.MX_WS_SCAN, c["rows"])),
                 ws_seg=_zeros(abi.mx_workspace_bytes(abi.MX_WS_SEGMENTED, values.numel())))
    elif kind == "matmul":
        A, B, gC = _matmul_inputs(c, seed)
        s.update(A=A, B=B, gC=gC, C=torch.empty_like(gC), gA=torch.empty_like(A), gB=torch.empty_like(B))
    elif kind == "dot":
        a, b, *g = _dot_inputs(c, seed)
        s.update(a=a, b=b, ws=_zeros(abi.mx_workspace_bytes(abi.MX_WS_REDUCE, c["len"])))
        if g:
            s.update(g=g[0], out=_empty(1), ga=torch.empty_like(a), gb=torch.empty_like(b))
        else:
            s.update(g=None, out=_empty(1, dtype=torch.int64))
    elif kind == "nbody":
        pos4, vel4 = _nbody_inputs(c, seed)
        s.update(pos4=pos4, vel4=vel4, ke=_empty(1), gx=torch.empty_like(pos4), gv=torch.empty_like(pos4),
                 ws=_zeros(abi.mx_nbody_workspace_bytes(c["n"], c["steps"], c["ckpt"])))
    elif kind == "kmeans":
        X, C, g = _kmeans_inputs(c, seed)
        s.update(X=X, C=C, g=g, labels=_empty(c["n"], dtype=torch.int32), counts=_empty(c["k"], dtype=torch.int64),
                 C_out=torch.empty_like(C), sse=_empty(1), gX=torch.empty_like(X),
                 ws=_zeros(abi.mx_kmeans_workspace_bytes(c["n"], c["d"], c["k"])), ws_sse=_zeros(256 + 4096))
    elif kind == "batch":
        table, A, B, gout = _batch_inputs(c, seed)
        s.update(batch=api.Batch(table), A=A, B=B, gout=gout, out=torch.zeros_like(gout), gA=torch.zeros_like(A),
                 gB=torch.zeros_like(B))
    elif kind == "body":
        a, b, g = _body_inputs(c, seed)
        x, y = api.body_inputs(2)
        d = x - y
        body = api.Body(api.exp(-(d * d)) * 0.5 + x * y, 2)
        s.update(body=body, a=a, b=b, g=g, out=_empty(1), ga=torch.empty_like(a), gb=torch.empty_like(b),
                 ws=_zeros(abi.mx_expr_workspace_bytes(body.e, c["n"])))
    else:
        k, phi, x = _mriq_inputs(c, seed)
        s.update(k=k, phi=phi, x=x, qr=_empty(c["voxels"]), qi=_empty(c["voxels"]))
    return s


def run(s):
    kind = s["kind"]
    if kind == "ragged":
        abi.mx_lengths_to_offsets(s["lengths"], s["off"], s["ws_scan"])
        abi.mx_segmented_reduce(s["op"], s["values"], s["off"], s["ne"], s["out"], s["ws_seg"])
        abi.mx_segmented_reduce_adjoint_f32(s["op"], s["values"], s["off"], s["ne"], s["gout"], s["gval"])
        return {"offsets": s["off"], "out": s["out"], "gvalues": s["gval"]}
    if kind == "matmul":
        abi.mx_map_map_reduce_f32(0, 0, s["A"], s["B"], s["C"])
        abi.mx_map_map_reduce_f32(0, 1, s["gC"], s["B"], s["gA"])
        abi.mx_map_map_reduce_f32(1, 0, s["A"], s["gC"], s["gB"])
        return {"C": s["C"], "gA": s["gA"], "gB": s["gB"]}
    if kind == "dot":
        abi.mx_map2_reduce(abi.MX_B_MUL, abi.MX_ADD, s["a"], s["b"], 0, s["out"], s["ws"])
        if s["g"] is None:
            return {"out": s["out"]}
        abi.mx_dot_adjoint_f32(s["a"], s["b"], s["g"], s["ga"], s["gb"])
        return {"out": s["out"], "ga": s["ga"], "gb": s["gb"]}
    if kind == "nbody":
        c = s["c"]
        abi.mx_nbody_ke_grad_f32(s["pos4"], s["vel4"], EPS2, G, DT, c["steps"], c["ckpt"], s["ke"], s["gx"], s["gv"],
                                 s["ws"])
        return {"ke": s["ke"], "gx": s["gx"], "gv": s["gv"]}
    if kind == "kmeans":
        abi.mx_kmeans_step_f32(s["X"], s["C"], s["labels"], s["counts"], s["C_out"], s["ws"])
        abi.mx_kmeans_sse_f32(s["X"], s["C_out"], s["labels"], s["sse"], s["ws_sse"])
        abi.mx_kmeans_sse_grad_f32(s["X"], s["C_out"], s["labels"], s["g"], s["gX"])
        return {"labels": s["labels"], "counts": s["counts"], "C": s["C_out"], "sse": s["sse"], "gX": s["gX"]}
    if kind == "batch":
        s["batch"].forward(s["A"], s["B"], s["out"])
        s["batch"].backward(s["A"], s["B"], s["gout"], s["gA"], s["gB"])
        return {"out": s["out"], "gA": s["gA"], "gB": s["gB"]}
    if kind == "body":
        xs, n = [s["a"], s["b"]], s["c"]["n"]
        abi.mx_expr_map_reduce(s["body"].e, abi.MX_ADD, xs, n, 0.0, s["out"], s["ws"])
        abi.mx_expr_vjp(s["body"].e, xs, n, None, s["g"], [s["ga"], s["gb"]])
        return {"out": s["out"], "ga": s["ga"], "gb": s["gb"]}
    abi.mx_mriq_f32(*s["k"], s["phi"], *s["x"], s["qr"], s["qi"])
    return {"qr": s["qr"], "qi": s["qi"]}


# ---------------------------------------------------------------- the least work of a pass
def work(case):
    c, kind = case, case["kind"]
    if kind == "ragged":
        # mean of the log-uniform lengths; the reverse of a sum needs no values
        nv = c["rows"] * 0.99 * (c["lmax"] / math.log(c["lmax"] + 1) - 0.5)
        return {"bytes": 4 * nv * 2 + c["rows"] * (8 + 8 + 4 + 4), "flops": nv}
    if kind == "matmul":
        m, n, k = c["m"], c["n"], c["k"]
        return {"bytes": 8 * (m * k + k * n + m * n), "flops": 6 * m * n * k}
    if kind == "dot":
        n = c["len"]
        return {"bytes": 16 * n, "flops": 4 * n} if c["dtype"] == "float32" else {"bytes": 8 * n, "flops": 2 * n}
    if kind == "nbody":
        # 20 flops a pair forward, 45 in the reverse, each step once
        return {"bytes": 64 * c["n"], "flops": 65.0 * c["steps"] * c["n"] ** 2}
    if kind == "kmeans":
        n, d, k = c["n"], c["d"], c["k"]
        return {"bytes": 8 * n * d + 4 * n + 8 * k * d + 8 * k, "flops": 2 * n * d * k + 5 * n * d}
    if kind == "batch":
        # mean of the log-uniform sizes; a dot reads and writes two such operands, a matvec one
        e = c["tasks"] * (c["smax"] - 100) / math.log(c["smax"] / 100)
        return {"bytes": 1.5 * 4 * 2 * e, "flops": 1.5 * 2 * e + 1.5 * e}
    if kind == "body":
        return {"bytes": 16 * c["n"], "flops": 20 * c["n"]}
    return {"bytes": 16 * c["samples"] + 20 * c["voxels"], "flops": 14 * c["samples"] * c["voxels"]}


# ---------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "ragged":
        lengths, values, gout = _ragged_inputs(c, seed)
        n, v = values.numel(), values.double()
        off = torch.zeros(c["rows"] + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(lengths, 0)
        row = torch.repeat_interleave(torch.arange(c["rows"], device=DEV), lengths)
        if c["op"] == "sum":
            out = torch.zeros(c["rows"], dtype=torch.float64, device=DEV).index_add_(0, row, v)
            return {"offsets": off, "out": out, "gvalues": gout.double()[row]}
        out = torch.full((c["rows"],), NE[c["op"]], dtype=torch.float64, device=DEV)
        out = out.scatter_reduce(0, row, v, "amax" if c["op"] == "max" else "amin")
        # the first element attaining the extreme takes the gradient
        at = torch.where(v == out[row], torch.arange(n, device=DEV), n)
        first = torch.full((c["rows"],), n, dtype=torch.int64, device=DEV).scatter_reduce(0, row, at, "amin")
        gval = torch.zeros(n + 1, dtype=torch.float64, device=DEV)
        gval[first] = gout.double()
        return {"offsets": off, "out": out, "gvalues": gval[:n]}
    if kind == "matmul":
        A, B, gC = (t.double() for t in _matmul_inputs(c, seed))
        return {"C": A @ B, "gA": gC @ B.t().contiguous(), "gB": A.t().contiguous() @ gC}
    if kind == "dot":
        a, b, *g = (t.double() for t in _dot_inputs(c, seed))
        if not g:
            return None
        return {"out": (a * b).sum().view(1), "ga": g[0] * b, "gb": g[0] * a}
    if kind == "nbody":
        return _nbody_exact(c, seed)
    if kind == "kmeans":
        X, C, g = (t.double() for t in _kmeans_inputs(c, seed))
        n, k = c["n"], c["k"]
        labels = torch.empty(n, dtype=torch.int64, device=DEV)
        step = max(1, (1 << 27) // (k * c["d"]))
        for p in range(0, n, step):
            labels[p:p + step] = ((X[p:p + step, None, :] - C[None]) ** 2).sum(-1).argmin(1)
        counts = torch.bincount(labels, minlength=k)
        sums = torch.zeros_like(C).index_add_(0, labels, X)
        new = torch.where(counts[:, None] > 0, sums / counts.clamp(min=1)[:, None], C)
        diff = X - new[labels]
        return {"labels": None, "counts": None, "C": new, "sse": (diff * diff).sum().view(1), "gX": 2 * g * diff}
    if kind == "batch":
        table, A, B, gout = _batch_inputs(c, seed)
        A, B, gout = A.double(), B.double(), gout.double()
        out, gA, gB = torch.zeros_like(gout), torch.zeros_like(A), torch.zeros_like(B)
        for kind_t, rows, cols, ao, bo, oo in table.tolist():
            a, b, go = A[ao:ao + rows * cols].view(rows, cols), B[bo:bo + cols], gout[oo:oo + rows]
            out[oo:oo + rows] = (a * b).sum(1)
            gA[ao:ao + rows * cols] = (go[:, None] * b[None]).reshape(-1)
            gB[bo:bo + cols] = (a * go[:, None]).sum(0)
        return {"out": out, "gA": gA, "gB": gB}
    if kind == "body":
        a, b, g = (t.double() for t in _body_inputs(c, seed))
        d = a - b
        e = 0.5 * torch.exp(-d * d)
        return {"out": (e + a * b).sum().view(1), "ga": g * (b - 2 * d * e), "gb": g * (a + 2 * d * e)}
    k, phi, x = _mriq_inputs(c, seed)
    k, x, phi = [t.double() for t in k], [t.double() for t in x], phi.double()
    qr, qi = (torch.empty(c["voxels"], dtype=torch.float64, device=DEV) for _ in range(2))
    for p in range(0, c["voxels"], 16384):
        t = sum(x[j][p:p + 16384, None] * k[j][None] for j in range(3)) * (2 * math.pi)
        qr[p:p + 16384], qi[p:p + 16384] = (torch.cos(t) * phi).sum(1), (torch.sin(t) * phi).sum(1)
    return {"qr": qr, "qi": qi}


def _nbody_exact(c, seed):
    """The loop and its reverse from the formulas, every state kept."""
    pos4, vel4 = _nbody_inputs(c, seed)
    x, v, m = pos4[:, :3].double(), vel4[:, :3].double(), pos4[:, 3].double()
    eps2, dt = float(np.float32(EPS2)), float(np.float32(DT))
    n, chunk = c["n"], max(1, (1 << 26) // c["n"])

    def accel(x):
        out = torch.empty_like(x)
        for p in range(0, n, chunk):
            d = x[None] - x[p:p + chunk, None]
            s = (d * d).sum(-1) + eps2
            out[p:p + chunk] = ((m * s ** -1.5)[..., None] * d).sum(1)
        return G * out

    def accel_vjp(x, ab):
        out = torch.empty_like(x)
        for p in range(0, n, chunk):
            d = x[None] - x[p:p + chunk, None]
            w = m[p:p + chunk, None, None] * ab[None] - m[None, :, None] * ab[p:p + chunk, None]
            s = (d * d).sum(-1) + eps2
            phi = s ** -1.5
            out[p:p + chunk] = (phi[..., None] * w - (3 * phi / s * (d * w).sum(-1))[..., None] * d).sum(1)
        return G * out

    states = []
    for _ in range(c["steps"]):
        states.append(x)
        x, v = x + dt * v, v + dt * accel(x)
    ke = (0.5 * m * (v * v).sum(1)).sum().view(1)
    xb, vb = torch.zeros_like(x), m[:, None] * v
    for x in reversed(states):
        xb, vb = xb + dt * accel_vjp(x, vb), vb + dt * xb
    pad = torch.zeros(n, 1, dtype=torch.float64, device=DEV)
    return {"ke": ke, "gx": torch.cat([xb, pad], 1), "gv": torch.cat([vb, pad], 1)}
