"""Map bodies at the edges of a block's chunk: one chunk is 4096 elements of float32 (2048 of float64, half of it for the
element-wise passes of three and four inputs), a single block reduces up to four chunks in one launch, and a pass larger
than the memory-side cache loads past it.  Unaligned slices take the same path."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import check_scalar, say
from test_gpu_expr import ALL_OPS, DEV, GAUSS_DOT, HORNER, IN, ND, OP, TD, U, X, _vjp_tol, check_map, error_bound, host

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi
FOUR = ([IN(0, 0), IN(1, 1), IN(2, 2), IN(3, 3), OP(X.MX_X_MUL, 0, 0, 1), OP(X.MX_X_ADD, 0, 0, 2),
         OP(X.MX_X_MUL, 0, 0, 3)], 4, 0)
PROGRAMS = {"one": HORNER, "two": GAUSS_DOT, "three": ALL_OPS, "four": FOUR}


def make(nin, n, dtype, seed, shift):
    rng = np.random.default_rng(seed)
    lo, hi = [-1, -1, 0.5, -1], [1, 1, 2.0, 1]
    xs = [rng.uniform(lo[k], hi[k], n).astype(ND[dtype]) for k in range(nin)]
    return xs, [slice_of(x, shift) for x in xs]


def slice_of(x, shift):
    big = torch.zeros(len(x) + shift, dtype=torch.from_numpy(x).dtype, device=DEV)
    big[shift:] = torch.from_numpy(x)
    return big[shift:]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 7, 1024, 2047, 2049, 4096, 8195, 16384, 16385, 20481])
@pytest.mark.parametrize("dtype", [abi.MX_F32, abi.MX_F64])
@pytest.mark.parametrize("name", list(PROGRAMS))
def test_chunk_edges(name, dtype, n, shift):
    prog, nin, out = PROGRAMS[name]
    say("expr chunk", name, dtype, n, shift)
    xs, ds = make(nin, n, dtype, n + nin, shift)
    e = abi.mx_expr_create(prog, nin, out, dtype)
    guard = torch.full((n + shift + 5,), 7.0, dtype=TD[dtype], device=DEV)
    abi.mx_expr_map(e, ds, guard[shift:shift + n])
    g = host(guard)
    check_map(g[shift:shift + n], prog, out, xs, dtype, f"{name} n={n}")
    assert np.all(g[:shift] == 7) and np.all(g[shift + n:] == 7)

    ws = torch.zeros(abi.mx_expr_workspace_bytes(e, n), dtype=torch.uint8, device=DEV)
    vals, bnd = O.expr_map(prog, out, *xs), 4 * error_bound(prog, out, xs, U[dtype])
    r = torch.empty((), dtype=TD[dtype], device=DEV)
    abi.mx_expr_map_reduce(e, abi.MX_ADD, ds, n, 0.25, r, ws)
    # the values' own bounds, and n + 1 additions of at most the absolute sum
    S = np.abs(vals).sum() + 0.25
    assert abs(float(host(r)) - (vals.sum() + 0.25)) <= bnd.sum() + (n + 1) * U[dtype] * S
    abi.mx_expr_map_reduce(e, abi.MX_MAX, ds, n, -9.0, r, ws)
    assert abs(float(host(r)) - vals.max()) <= bnd.max()

    rng = np.random.default_rng(n)
    gout = rng.uniform(-1, 1, n).astype(ND[dtype])
    grads = [torch.full((n + shift + 5,), 7.0, dtype=TD[dtype], device=DEV) for _ in range(nin)]
    abi.mx_expr_vjp(e, ds, n, slice_of(gout, shift), None, [t[shift:shift + n] for t in grads])
    ref = O.expr_vjp(prog, out, xs, gout=gout, gscale=None)
    for k in range(nin):
        h = host(grads[k]).astype(np.float64)
        scale = np.linalg.norm(ref[k]) / np.sqrt(n) + 1e-300
        assert np.all(np.abs(h[shift:shift + n] - ref[k]) <= _vjp_tol(dtype) * (np.abs(ref[k]) + scale)), k
        assert np.all(h[:shift] == 7) and np.all(h[shift + n:] == 7)


def test_in_place_map_and_gradient():
    """Outputs over the inputs: a group is loaded whole before it is stored."""
    prog, nin, out = GAUSS_DOT
    n = 3 * 4096 + 5
    say("expr in place", n)
    xs, ds = make(nin, n, abi.MX_F32, 3, 0)
    e = abi.mx_expr_create(prog, nin, out, abi.MX_F32)
    ref = [torch.empty_like(d) for d in ds]
    abi.mx_expr_vjp(e, ds, n, None, None, ref)
    mapped = torch.empty_like(ds[0])
    abi.mx_expr_map(e, ds, mapped)
    a = [d.clone() for d in ds]
    abi.mx_expr_map(e, a, a[1])
    assert torch.equal(a[1], mapped)
    b = [d.clone() for d in ds]
    abi.mx_expr_vjp(e, b, n, None, None, [b[1], b[0]])
    assert torch.equal(b[1], ref[0]) and torch.equal(b[0], ref[1])


def test_past_the_cache():
    """Five arrays of 64 MiB: loads past the caches, the remainders in the last block."""
    prog, nin, out = FOUR
    n = (1 << 24) + 1027
    say("expr past the cache", n)
    xs, ds = make(nin, n, abi.MX_F32, 9, 1)
    e = abi.mx_expr_create(prog, nin, out, abi.MX_F32)
    o = torch.empty(n, device=DEV)
    abi.mx_expr_map(e, ds, o)
    check_map(host(o), prog, out, xs, abi.MX_F32, "past the cache")
    grads = [torch.full((n,), np.nan, device=DEV) for _ in range(nin)]
    abi.mx_expr_vjp(e, ds, n, None, None, grads)
    a, b, c, d = (x.astype(np.float64) for x in xs)
    for g, r in zip(grads, (b * d, a * d, d, a * b + c)):
        h = host(g).astype(np.float64)
        assert np.all(np.abs(h - r) <= 2e-5 * (np.abs(r) + np.linalg.norm(r) / np.sqrt(n)))
    ws = torch.zeros(abi.mx_expr_workspace_bytes(e, n), dtype=torch.uint8, device=DEV)
    r = torch.empty((), device=DEV)
    abi.mx_expr_map_reduce(e, abi.MX_ADD, ds, n, 0.0, r, ws)
    v = (a * b + c) * d
    check_scalar(float(host(r)), float(v.sum()), float(np.abs(v).sum()), n, what="past the cache")


@pytest.mark.parametrize("vectors,more", [(511, 3), (512, 0), (513, 1), (1 << 17, 0), ((1 << 17) + 1, 1), ((1 << 17) + 1500, 3)])
@pytest.mark.parametrize("dtype", [abi.MX_F32, abi.MX_F64])
@pytest.mark.parametrize("name", ["two", "four"])
def test_small_pass_edges(name, dtype, vectors, more):
    """Passes of one vector per thread, up to 2^17 vectors, and the first past them."""
    width = 4 if dtype == abi.MX_F32 else 2
    test_chunk_edges(name, dtype, vectors * width + more % width, 1)


@pytest.mark.parametrize("vectors,more", [(255, 1), (1023, 0), (1024, 3), (1025, 0), (4095, 1), (4096, 3), (4097, 0), (8193, 1)])
@pytest.mark.parametrize("dtype", [abi.MX_F32, abi.MX_F64])
@pytest.mark.parametrize("name", ["one", "four"])
def test_one_block(name, dtype, vectors, more):
    """Sums of one block of 256 threads (1024 vectors), of 1024 (4096), and of two launches."""
    test_small_pass_edges(name, dtype, vectors, more)
