"""Batches at the edges of their tiles: rows of every length modulo four around what a block takes at once, rows past the
LDS copy of x and past what a 32-bit offset reaches, dots around a backward tile, unaligned offsets with gaps that must stay
untouched, several configurations, and a batch larger than the memory-side cache."""
import numpy as np
import pytest
import torch

from parity import say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
api = mx.api
U = 2.0 ** -24


def layout(tasks, gap, a0=0):
    """(kind, rows, cols) -> the plan's table, operands apart by `gap` floats; and the lengths of A, B and out."""
    tb, a, b, o = [], a0, gap, 0
    for kind, rows, cols in tasks:
        tb.append((kind, rows, cols, a, b, o))
        a, b, o = a + rows * cols + gap, b + cols + gap, o + rows + 1
    return np.array(tb, np.int64), a, b, o


def check(tasks, cfg, gap, a0=0):
    tb, na, nb, no = layout(tasks, gap, a0)
    g = torch.Generator(device="cuda").manual_seed(len(tasks) + gap)
    A, B, gout = (torch.rand(n, device="cuda", generator=g) * 2 - 1 for n in (na, nb, no))
    out, gA, gB = (torch.full((n,), 7.0, device="cuda") for n in (no, na, nb))
    batch = api.Batch(tb, cfg)
    batch.forward(A, B, out)
    batch.backward(A, B, gout, gA, gB)
    torch.cuda.synchronize()
    h = {k: v.cpu().numpy() for k, v in dict(A=A, B=B, gout=gout, out=out, gA=gA, gB=gB).items()}
    used = {k: np.zeros(len(h[k]), bool) for k in ("out", "gA", "gB")}
    for kind, rows, cols, a, b, o in tb:
        M = h["A"][a:a + rows * cols].reshape(rows, cols)
        x, gr = h["B"][b:b + cols], h["gout"][o:o + rows]
        M64, x64, g64 = M.astype(np.float64), x.astype(np.float64), gr.astype(np.float64)
        what = (kind, rows, cols, cfg, gap)
        err = np.abs(h["out"][o:o + rows] - M64 @ x64)
        assert np.all(err <= (cols + 2) * U * (np.abs(M64) @ np.abs(x64))), what
        # one product per element
        assert np.array_equal(h["gA"][a:a + rows * cols].reshape(rows, cols), gr[:, None] * x[None]), what
        err = np.abs(h["gB"][b:b + cols] - g64 @ M64)
        assert np.all(err <= (rows + 2) * U * (np.abs(g64) @ np.abs(M64))), what
        used["out"][o:o + rows] = used["gA"][a:a + rows * cols] = used["gB"][b:b + cols] = True
    for k, m in used.items():
        assert np.all(h[k][~m] == 7.0), (k, cfg, gap)


COLS = [1, 2, 3, 4, 5, 6, 7, 15, 63, 64, 65, 66, 127, 128, 129, 130, 255, 256, 257, 259, 511, 513, 682, 683, 1000, 1023,
        1025, 1366, 2047, 2048, 2049, 2050, 4099]
DOTS = [0, 1, 3, 4, 5, 1023, 4095, 4096, 4097, 8191, 8195, 16384, 16387, 40001]


@pytest.mark.parametrize("gap", [0, 1, 3])
@pytest.mark.parametrize("cfg", [None, (4096, 8), (5001, 2), (16384, 1), (65536, 16)])
def test_edges(cfg, gap):
    say("batch tiles", cfg, gap)
    tasks = [(1, rows, c) for c in COLS for rows in (1, 7, 17, 70)] + [(0, 1, n) for n in DOTS]
    tasks += [(1, 9000, 3), (1, 5000, 6), (1, 0, 40), (1, 3, 0)]
    check(tasks, cfg, gap)


@pytest.mark.parametrize("gap", [0, 1])
def test_long_rows(gap):
    """A row past the 32-bit offset's reach goes alone; a shorter long row does not."""
    say("batch long rows", gap)
    check([(1, 3, (1 << 22) + 3), (1, 3, (1 << 21) + 1), (1, 1, (1 << 22) + 4)], None, gap)


def test_past_the_cache():
    """A table whose operands lie further apart than the memory-side cache."""
    say("batch past the cache")
    check([(1, 40, 1001), (1, 100, 64), (0, 1, 100003), (1, 5, 3)], None, 1, a0=34 << 20)


@pytest.mark.parametrize("gap", [0, 1])
def test_no_rows(gap):
    """A matvec of no rows, of one pass over the columns to many: gx is zero and nothing else is written, whatever lies
    behind it in the pools."""
    say("batch no rows", gap)
    cols = [0, 3, 4, 7, 2047, 2048, 2049, 2052, 4096, 4099, (1 << 22) + 3]
    tasks = [t for c in cols for t in ((1, 0, c), (1, 9, 2049))] + [(0, 1, 9000)]
    check(tasks, None, gap)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_x(value):
    """A non-finite element of x reaches each row by one product, whichever element it is: the lanes past a row's end
    add nothing."""
    say("batch non-finite x", value)
    cols = [1, 2, 3, 5, 6, 7, 63, 65, 66, 67, 127, 129, 130, 131, 191, 255, 257, 259, 301, 514, 1001, 2045, 2046, 2047,
            2049, 4099]
    tasks = [(1, 21, c) for c in cols for _ in range(3)] + [(0, 1, c) for c in cols]
    tb, na, nb, no = layout(tasks, 0)
    A, B = (np.random.default_rng(5).uniform(0.5, 1.0, n).astype(np.float32) for n in (na, nb))
    A *= np.random.default_rng(6).choice([-1, 1], na).astype(np.float32)
    for i, (_, _, c, _, b, _) in enumerate(tb):
        B[b + (c - 1, 0, c // 2)[i % 3]] = value
    out = torch.empty(no, device="cuda")
    api.Batch(tb).forward(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), out)
    h = out.cpu().numpy()
    for _, rows, c, a, b, o in tb:
        ref = (A[a:a + rows * c].reshape(rows, c).astype(np.float64) * B[b:b + c]).sum(1)
        assert np.array_equal(h[o:o + rows], ref.astype(np.float32), equal_nan=True), (rows, c)


def test_autotune_times_each_launch_once():
    """More than eight blocks per CU are the launches of eight: the tuner does not choose between them."""
    say("batch autotune candidates")
    tb, na, nb, no = layout([(0, 1, 20000), (1, 100, 300)] * 20, 0)
    A, B, gout, gA, gB, out = (torch.rand(n, device="cuda") for n in (na, nb, no, na, nb, no))
    for _ in range(3):
        assert api.Batch(tb).autotune(A, B, out, gout, gA, gB)[1] in (2, 4, 8)


@pytest.mark.parametrize("gap", [0, 1])
@pytest.mark.parametrize("cfg", [None, (65536, 8), (4096, 2)])
def test_wide_and_tall_backward(cfg, gap):
    """Long rows in several tiles of columns (remainders of one to four past 2048), short ones whose many phases are added
    in parts, rows of one to three elements in several rounds, and tasks of many tiles whose sums are added in runs."""
    say("batch wide and tall", cfg, gap)
    tasks = [(1, r, c) for c in (2051, 2052, 4095, 4096, 4097, 4098, 4100, 6145, 20003) for r in (1, 2, 9, 20)]
    tasks += [(1, r, c) for c in (1, 2, 3, 4, 5, 17, 33) for r in (1, 2, 15, 17, 511, 2049, 4097, 8193)]
    tasks += [(1, 40000, 1), (1, 30000, 4), (1, 3000, 1001), (1, 700, 2100)]
    check(tasks, cfg, gap)
