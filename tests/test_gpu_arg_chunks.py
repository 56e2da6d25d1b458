"""The reverse of a min / max at the edges of a block's chunk (4096 elements), unaligned: the gradient at the first of
equal extremes, zeros everywhere else, nothing written outside."""
import numpy as np
import pytest
import torch

from parity import say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 4, 1023, 4095, 4096, 4097, 8195, 65537, (1 << 22) + 4101])
@pytest.mark.parametrize("op", [abi.MX_MIN, abi.MX_MAX])
def test_arg_chunks(op, n, shift):
    say("arg chunk", op, n, shift)
    rng = np.random.default_rng(n)
    x = rng.integers(-9, 10, n).astype(np.float32)  # many equal extremes
    places = {0, n - 1, n // 2, (n // 4096) * 4096 - 1, (n // 4) * 4}
    for at in sorted(p for p in places if 0 <= p < n):
        y = x.copy()
        y[at] = 20.0 if op == abi.MX_MAX else -20.0
        for v in (x, y):
            d = torch.zeros(n + shift, device="cuda")
            d[shift:] = torch.from_numpy(v)
            big = torch.full((n + shift + 5,), 7.0, device="cuda")
            ws = torch.zeros(abi.mx_workspace_bytes(abi.MX_WS_REDUCE, n, 0), dtype=torch.uint8, device="cuda")
            ne = -100.0 if op == abi.MX_MAX else 100.0
            abi.mx_reduce_adjoint_f32(op, d[shift:], ne, torch.tensor([0.5], device="cuda"), big[shift:shift + n], ws)
            ref = np.zeros(n, np.float32)
            ref[v.argmax() if op == abi.MX_MAX else v.argmin()] = 0.5
            h = big.cpu().numpy()
            assert np.array_equal(h[shift:shift + n], ref), (op, n, at)
            assert np.all(h[:shift] == 7) and np.all(h[shift + n:] == 7)


@pytest.mark.parametrize("n", [2047, 2049, (1 << 19) - 1, (1 << 19) + 3, (1 << 19) + 4])
def test_small_pass_edges(n):
    """Chunks of 256 vectors up to 2^17 of them, and the first past it."""
    test_arg_chunks(abi.MX_MAX, n, 1)
