"""map, map2, the dot's adjoint and the reductions at the edges of a block's chunk (one to four vectors per thread, the
change between them at 2^16 vectors), of what a single block reduces alone, and past the memory-side cache; unaligned
slices; nothing written outside.  References in numpy: integer and single-operation float results are exact."""
import numpy as np
import pytest
import torch

from parity import say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi
TYPES = {"f32": (np.float32, np.float32), "f64": (np.float64, np.float64), "i32": (np.int32, np.int64),
         "i64": (np.int64, np.int64)}


def slice_of(x, shift):
    t = torch.zeros(len(x) + shift, dtype=torch.from_numpy(x[:0]).dtype, device="cuda")
    t[shift:] = torch.from_numpy(x)
    return t[shift:]


def guarded(n, dtype, shift):
    t = torch.full((n + shift + 5,), 7, dtype=torch.from_numpy(np.zeros(0, dtype)).dtype, device="cuda")
    return t, t[shift:shift + n]


def whole(t, n, shift):
    torch.cuda.synchronize()
    h = t.cpu().numpy()
    assert np.all(h[:shift] == 7) and np.all(h[shift + n:] == 7)
    return h[shift:shift + n]


def make(kind, n, seed):
    rng = np.random.default_rng(seed)
    t = TYPES[kind][0]
    return (rng.uniform(-1, 1, n) if kind[0] == "f" else rng.integers(-10 ** 6, 10 ** 6, n)).astype(t)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 255, 1023, 1025, 4096, 4099, 16384, 16387, 32771, (1 << 17) + 1, (1 << 18) + 3,
                               (1 << 18) + 4099])
@pytest.mark.parametrize("kind", list(TYPES))
def test_chunk_edges(kind, n, shift):
    say("stream chunk", kind, n, shift)
    acc = TYPES[kind][1]
    a, b = make(kind, n, n), make(kind, n, n + 1)
    da, db = slice_of(a, shift), slice_of(b, shift)
    wide_a, wide_b = a.astype(acc), b.astype(acc)
    t, o = guarded(n, acc, shift)
    abi.mx_map(abi.MX_U_SQ, da, None, o)
    assert np.array_equal(whole(t, n, shift), wide_a * wide_a)
    t, o = guarded(n, acc, shift)
    abi.mx_map2(abi.MX_B_SUB, da, db, o)
    assert np.array_equal(whole(t, n, shift), wide_a - wide_b)

    ws = torch.zeros(abi.mx_workspace_bytes(abi.MX_WS_REDUCE, n, 0), dtype=torch.uint8, device="cuda")
    r = torch.zeros(1, dtype=o.dtype, device="cuda")
    ne = 3 if kind[0] == "i" else 0.25
    for op, ref in ((abi.MX_MIN, lambda x: min(ne, x.min())), (abi.MX_MAX, lambda x: max(ne, x.max()))):
        abi.mx_reduce(op, da, ne, r, ws)
        assert r.cpu().numpy()[0] == acc(ref(wide_a))
    abi.mx_reduce(abi.MX_ADD, da, ne, r, ws)
    abi.mx_map2_reduce(abi.MX_B_MUL, abi.MX_ADD, da, db, ne, (d := torch.zeros_like(r)), ws)
    got_sum, got_dot = r.cpu().numpy()[0], d.cpu().numpy()[0]
    if kind[0] == "i":
        assert got_sum == wide_a.sum() + ne and got_dot == (wide_a * wide_b).sum() + ne
    else:
        u = 2.0 ** -24 if kind == "f32" else 2.0 ** -53
        a64, b64 = a.astype(np.longdouble), b.astype(np.longdouble)
        assert abs(got_sum - (a64.sum() + ne)) <= (n + 1) * u * (np.abs(a64).sum() + ne)
        assert abs(got_dot - ((a64 * b64).sum() + ne)) <= (n + 2) * u * (np.abs(a64 * b64).sum() + ne)

    if kind == "f32":
        g = torch.tensor([0.75], device="cuda")
        for want_a, want_b in ((1, 1), (1, 0), (0, 1)):
            (ta, ga), (tb, gb) = guarded(n, np.float32, shift), guarded(n, np.float32, shift)
            abi.mx_dot_adjoint_f32(da, db, g, ga if want_a else None, gb if want_b else None)
            if want_a:
                assert np.array_equal(whole(ta, n, shift), np.float32(0.75) * b)
            if want_b:
                assert np.array_equal(whole(tb, n, shift), np.float32(0.75) * a)


def test_in_place():
    """map2 over its own operand and map over its input."""
    n = (1 << 18) + 4099
    say("stream in place", n)
    a, b = make("f32", n, 1), make("f32", n, 2)
    da, db = slice_of(a, 0), slice_of(b, 0)
    abi.mx_map2(abi.MX_B_ADD, da, db, db)
    assert np.array_equal(db.cpu().numpy(), a + b)
    abi.mx_map(abi.MX_U_SQ, da, None, da)
    assert np.array_equal(da.cpu().numpy(), a * a)


@pytest.mark.parametrize("kind", ["f32", "i32"])
def test_past_the_cache(kind):
    """More than 256 MiB in a pass."""
    n = (34 << 20) + 3
    say("stream past the cache", kind, n)
    acc = TYPES[kind][1]
    a, b = make(kind, n, 5), make(kind, n, 6)
    da, db = slice_of(a, 1), slice_of(b, 1)
    t, o = guarded(n, acc, 1)
    abi.mx_map2(abi.MX_B_MUL, da, db, o)
    assert np.array_equal(whole(t, n, 1), a.astype(acc) * b.astype(acc))
    t, o = guarded(n, acc, 1)
    abi.mx_map(abi.MX_U_NEG, da, None, o)
    assert np.array_equal(whole(t, n, 1), -a.astype(acc))
    if kind == "f32":
        g = torch.tensor([-1.5], device="cuda")
        (ta, ga), (tb, gb) = guarded(n, np.float32, 1), guarded(n, np.float32, 1)
        abi.mx_dot_adjoint_f32(da, db, g, ga, gb)
        assert np.array_equal(whole(ta, n, 1), np.float32(-1.5) * b) and np.array_equal(whole(tb, n, 1), np.float32(-1.5) * a)


@pytest.mark.parametrize("n", [(1 << 19) - 1, (1 << 19) + 3, (1 << 19) + 4099, (1 << 21) - 1, (1 << 21) + 5, (1 << 23) - 3,
                               (1 << 23) + 3, (1 << 25) - 1])
@pytest.mark.parametrize("kind", ["f32", "i32", "f64"])
def test_read_back(kind, n):
    """On both sides of the passes' one vector per thread (2^17 vectors) and of each way of storing (16 MB, half the
    memory-side cache and all of it): a pass reduced by the next, in place, and the dot's adjoint; nothing outside."""
    say("stream read back", kind, n)
    acc = TYPES[kind][1]
    a, b = make("i32", n, 8) % 1000, make("i32", n, 9) % 1000  # whole numbers: every result and sum below 2^53 is exact
    a, b = a.astype(TYPES[kind][0]), b.astype(TYPES[kind][0])
    da, db = slice_of(a, 1), slice_of(b, 1)
    t, o = guarded(n, acc, 1)
    ws = torch.zeros(abi.mx_workspace_bytes(abi.MX_WS_REDUCE, n, 0), dtype=torch.uint8, device="cuda")
    r = torch.zeros(2, dtype=o.dtype, device="cuda")
    abi.mx_map2(abi.MX_B_SUB, da, db, o)
    abi.mx_reduce(abi.MX_MAX, o, -5000, r[:1], ws)
    if kind == "f32":
        abi.mx_map(abi.MX_U_SQ, o, None, o)
    else:
        abi.mx_map2(abi.MX_B_MUL, o, o, o)
    abi.mx_reduce(abi.MX_ADD, o, 0, r[1:], ws)
    want = a.astype(acc) - b.astype(acc)
    got = r.cpu().numpy()
    assert got[0] == want.max()
    want = want * want
    assert np.array_equal(whole(t, n, 1), want)
    total = want.astype(np.float64).sum() if kind[0] == "f" else want.sum()
    if kind == "f32":  # a chain of at most n additions
        assert abs(got[1] - total) <= n * 2.0 ** -24 * total
    else:
        assert got[1] == total
    if kind == "f32":
        g = torch.tensor([0.5], device="cuda")
        (ta, ga), (tb, gb) = guarded(n, np.float32, 1), guarded(n, np.float32, 1)
        abi.mx_dot_adjoint_f32(da, db, g, ga, gb)
        assert np.array_equal(whole(ta, n, 1), np.float32(0.5) * b) and np.array_equal(whole(tb, n, 1), np.float32(0.5) * a)


@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("vectors", [255, 256, 257, 1023, 1024, 1025, 2048, 4095, 4096, 4097, 8193])
@pytest.mark.parametrize("kind", list(TYPES))
def test_one_block(kind, vectors, more):
    """Reductions of one block of 256 threads (1024 vectors), of 1024 (4096), and of two launches."""
    test_chunk_edges(kind, vectors * (2 if kind.endswith("64") else 4) + more, 1)
