"""The ragged reduce and its reverses by lane groups: every choice of group and of loads in flight, rows at the edges of
what a group takes alone, long rows among short ones, unaligned values; and the chunked kernels on the short rows that
small inputs no longer bring there."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import check_vector, say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi
NE = {abi.MX_ADD: 0, abi.MX_MUL: 1, abi.MX_MIN: 2 ** 63 - 1, abi.MX_MAX: -2 ** 63}
EDGES = [0, 1, 2, 3, 4, 5, 15, 16, 17, 127, 128, 129, 255, 256, 257, 258, 511, 512, 513, 514, 1023, 1024, 1025, 1026, 2047,
         2049, 4096, 4099]


def lengths(case):
    rng = np.random.default_rng(len(case))
    if case == "small_wave":        # up to 131 072 values, a wave per row, edges of a group's own rows
        return np.array(EDGES + [0, 0] + EDGES[::-1])
    if case == "small_lanes":       # 16 lanes per row; rows past 256 taken by the block
        L = rng.integers(0, 60, 3000)
        L[[5, 6, 900, 2999]] = [256, 257, 9000, 255]
        return L
    if case == "one_small_row":
        return np.array([131072])
    if case == "just_small":        # the last input of the small path, ragged in its last block
        L = np.full(1001, 130)
        L[-1] = 131072 - int(L[:-1].sum())
        return L
    if case == "many_lanes4":       # mean up to 48
        L = rng.integers(0, 80, 20001)
        L[::997] = 257
        L[7], L[20000] = 30000, 300
        return L
    if case == "many_lanes8":       # mean 48 .. 100
        L = rng.integers(0, 150, 9001)
        L[::503] = rng.choice(EDGES, len(L[::503]))
        L[8999] = 60000
        return L
    if case == "many_wave":         # mean 100 .. 300, up to 32 768 rows
        L = rng.integers(0, 400, 8200)
        L[::100] = rng.choice(EDGES, 82)
        L[4000] = 50001
        return L
    # chunked: fewer than 8192 rows, more than 131 072 values, thousands of rows in a chunk
    L = rng.integers(0, 4, 8000)
    L[4000], L[-1] = 140000, 4097
    return L


CASES = ["small_wave", "small_lanes", "one_small_row", "just_small", "many_lanes4", "many_lanes8", "many_wave", "chunked"]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("dt", [np.float32, np.float64, np.int32, np.int64])
def test_group_reduce(case, dt):
    say("ragged groups", case, np.dtype(dt).name)
    L = lengths(case).astype(np.int64)
    off = O.offsets_from_lengths(L)
    nv = int(off[-1])
    rng = np.random.default_rng(3)
    integer = np.issubdtype(dt, np.integer)
    ws = torch.zeros(abi.mx_workspace_bytes(abi.MX_WS_SEGMENTED, nv), dtype=torch.uint8, device="cuda")
    toff = torch.from_numpy(off).to("cuda")
    for op in NE if integer else [abi.MX_ADD, abi.MX_MAX]:
        if integer:
            v = rng.integers(-2, 3, nv).astype(dt) if op == abi.MX_MUL else rng.integers(-10 ** 6, 10 ** 6, nv).astype(dt)
            ne = NE[op]
        else:
            v, ne = rng.uniform(-1, 1, nv).astype(dt), 0.25 if op == abi.MX_ADD else -np.inf
        for shift in (0, 1):
            full = torch.from_numpy(np.concatenate([np.zeros(shift, dtype=dt), v])).to("cuda")
            out = torch.full((len(L),), 9, dtype=mx.api.ACC_OF[full.dtype], device="cuda")
            abi.mx_segmented_reduce(op, full[shift:], toff, ne, out, ws)
            got = out.cpu().numpy()
            R = O.segmented_reduce(op, ne, v, off)
            if integer or op == abi.MX_MAX:
                assert np.array_equal(got, R.astype(got.dtype)), (op, shift)
            else:
                check_vector(got, R, O.segmented_reduce(O.ADD, 0.25, np.abs(v), off), L + 1, what=f"{case} {shift}")
    assert not ws.any()


@pytest.mark.parametrize("case", CASES)
def test_group_reverses(case):
    say("ragged group reverses", case)
    L = lengths(case).astype(np.int64)
    off = O.offsets_from_lengths(L)
    nv = int(off[-1])
    rng = np.random.default_rng(4)
    # few distinct values: ties; a NaN here and there, which is never chosen
    v = rng.integers(-3, 4, nv).astype(np.float32)
    v[rng.integers(0, nv, 20)] = np.nan
    g = rng.uniform(-1, 1, len(L)).astype(np.float32)
    tg, toff = torch.from_numpy(g).to("cuda"), torch.from_numpy(off).to("cuda")
    for shift in (0, 1):
        full = torch.from_numpy(np.concatenate([np.zeros(shift, dtype=np.float32), v])).to("cuda")
        gv = torch.full((nv + 2,), 5.0, device="cuda")
        for op, ne in [(abi.MX_ADD, 0.0), (abi.MX_MIN, np.inf), (abi.MX_MAX, -np.inf), (abi.MX_MAX, 3.0),
                       (abi.MX_MIN, np.nan)]:
            gv.fill_(5.0)
            abi.mx_segmented_reduce_adjoint_f32(op, full[shift:], toff, ne, tg, gv[shift:nv + shift])
            got = gv.cpu().numpy()
            if op == abi.MX_ADD:
                ref = O.segmented_sum_adjoint(g, off)
            else:
                ref = O.segmented_reduce_adjoint(op, ne, v, off, g)
            assert np.array_equal(got[shift:nv + shift], ref.astype(np.float32)), (op, ne, shift)
            assert (got[:shift] == 5.0).all() and (got[nv + shift:] == 5.0).all()


LONG = {
    # many long rows to a block, for its waves in turn, and some past what a wave takes; sixteen lanes a row
    "lanes": np.array(([3] * 20 + [257, 300, 1025, 4096, 4097] + [0]) * 25 + [9] * 400 + [7000]),
    # a wave a row, and one or two long rows in a block, which takes them whole
    "wave": np.array([60] * 15 + [1025] + [70] * 14 + [1026, 16385] + [0, 50, 4097, 4099, 1500, 2000, 3000, 16384, 16385]),
    # as many rows as take sixteen lanes in the reverse of a maximum, twenty of them for their whole wave
    "reverse": np.array(([5] * 60 + [1024, 1025, 1029, 9001]) * 20),
}


@pytest.mark.parametrize("case", list(LONG))
@pytest.mark.parametrize("dt", [np.float32, np.float64, np.int32])
def test_long_rows_by_waves_and_blocks(case, dt, monkeypatch):
    monkeypatch.setitem(globals(), "lengths", LONG.__getitem__)
    test_group_reduce(case, dt)
    if dt == np.float32:
        test_group_reverses(case)


FEW_LONG = {
    # rows past a group on average, one to a block: by its first wave, by the whole block, empty ones, a single row
    "few": np.array([0, 3000, 1, 1024, 1025, 4097, 0, 9001, 511, 513, 6000, 2049]),
    "even": np.full(16, 6000),
    "single": np.array([1025]),
    # at that line for vectors of four and of two, and just below it
    "line4": np.array([1024, 1024, 1025]), "below4": np.array([1024, 1024, 1024]),
    "line2": np.array([512, 512, 513]), "below2": np.array([512, 512, 512]),
}


@pytest.mark.parametrize("case", list(FEW_LONG))
@pytest.mark.parametrize("dt", [np.float32, np.float64, np.int32, np.int64])
def test_few_long_rows(case, dt, monkeypatch):
    monkeypatch.setitem(globals(), "lengths", FEW_LONG.__getitem__)
    test_group_reduce(case, dt)
