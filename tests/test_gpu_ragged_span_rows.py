"""The row-span reduce and broadcast at every choice of rows per block (one to sixteen, eight of eight-byte sums and of
long rows), ragged last blocks, empty rows, rows that cross a wave's quarter, unaligned values."""
import numpy as np
import pytest
import torch

from parity import say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi


def slice_of(x, shift):
    t = torch.zeros(len(x) + shift, dtype=torch.from_numpy(x[:0]).dtype, device="cuda")
    t[shift:] = torch.from_numpy(x)
    return t[shift:]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("nseg,mean", [(8192, 310), (10003, 900), (20001, 330), (32769, 310), (40001, 130), (40007, 310),
                                       (33000, 640)])
@pytest.mark.parametrize("kind", ["f32", "i32"])
def test_rows_per_block(kind, nseg, mean, shift):
    say("ragged span rows", kind, nseg, mean, shift)
    rng = np.random.default_rng(nseg + mean)
    L = rng.integers(0, 2 * mean, nseg)
    L[::37] = 0
    L[5], L[nseg - 1], L[nseg // 2] = 9001, 4097, 16384
    off = np.concatenate([[0], np.cumsum(L)]).astype(np.int64)
    nv = int(off[-1])
    v = rng.uniform(-1, 1, nv).astype(np.float32) if kind == "f32" else rng.integers(-10 ** 6, 10 ** 6, nv).astype(np.int32)
    acc = np.float32 if kind == "f32" else np.int64
    ws = torch.zeros(abi.mx_workspace_bytes(abi.MX_WS_SEGMENTED, nv, 0), dtype=torch.uint8, device="cuda")
    dv, do = slice_of(v, shift), torch.from_numpy(off).cuda()
    out = torch.zeros(nseg, dtype=torch.from_numpy(np.zeros(0, acc)).dtype, device="cuda")
    abi.mx_segmented_reduce(abi.MX_ADD, dv, do, 0, out, ws)
    got = out.cpu().numpy()
    wide = v.astype(np.float64 if kind == "f32" else np.int64)
    csum = np.concatenate([[0], np.cumsum(wide.astype(np.longdouble) if kind == "f32" else wide)])
    ref = csum[off[1:]] - csum[off[:-1]]
    if kind == "i32":
        assert np.array_equal(got, ref)
    else:
        mag = np.concatenate([[0], np.cumsum(np.abs(wide))])
        mag = mag[off[1:]] - mag[off[:-1]]
        assert np.all(np.abs(got - ref) <= (L + 8) * 2.0 ** -24 * mag + 1e-12)
    ne = -2.0 if kind == "f32" else -2 ** 40
    abi.mx_segmented_reduce(abi.MX_MAX, dv, do, ne, out, ws)
    got = out.cpu().numpy()
    full = L > 0
    ref = np.full(nseg, ne, acc)
    ref[full] = np.maximum(np.maximum.reduceat(v.astype(acc), off[:-1][full]), acc(ne))
    assert np.array_equal(got, ref)
    if kind == "f32":
        g = rng.uniform(-1, 1, nseg).astype(np.float32)
        big = torch.full((nv + shift + 5,), 7.0, device="cuda")
        abi.mx_segmented_reduce_adjoint_f32(abi.MX_ADD, dv, do, 0.0, torch.from_numpy(g).cuda(), big[shift:shift + nv])
        h = big.cpu().numpy()
        assert np.array_equal(h[shift:shift + nv], np.repeat(g, L))
        assert np.all(h[:shift] == 7) and np.all(h[shift + nv:] == 7)
