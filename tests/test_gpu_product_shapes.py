"""Every tile shape of the dense product at the edges of its tiles, of its slices of K (32, dealt to groups of waves) and
on operands at 4-byte alignment, against the oracle; the sizes that are routed away from vectors of rows; K = 0."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from parity import check_vector, say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi

SHAPES = ["16x16", "32x32", "32x64", "64x32", "64x64", "80x64", "64x80", "96x64", "64x96", "128x64", "64x128", "128x96",
          "128x128", "128x128w16"]


def placed(x, shift):
    """x on the device, its first element `shift` floats past a 256-byte boundary, NaN around it."""
    buf = torch.full((x.size + 64 + shift,), float("nan"), device="cuda")
    v = buf[shift:shift + x.size].view(*x.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return v


def check(M, N, K, ta, tb, shift, what):
    say("product", what, M, N, K, ta, tb, shift)
    A, B = W.dense_f32(M, N, K, seed=M + 3 * N + 7 * K)
    C = torch.full((M, N), 7.0, device="cuda")
    abi.mx_map_map_reduce_f32(ta, tb, placed(A.T if ta else A, shift), placed(B.T if tb else B, shift), C)
    got, ref, S = C.cpu().numpy(), O.matmul(A, B), O.matmul(np.abs(A), np.abs(B))
    check_vector(got.ravel(), ref.ravel(), S.ravel(), K, what=f"{what} {M}x{N}x{K} {ta}{tb}")


@pytest.mark.parametrize("name", SHAPES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_product_shape_edges(name, ta, tb, monkeypatch):
    monkeypatch.setenv("MX_GEMM_TILE", name)
    bm, bn = (int(v) for v in name.replace("w16", "").split("x"))
    # one slice and less, slice edges, one to several rounds of slices for every group; below, at and past a tile
    for M, N, K, shift in [(bm, bn, 32, 0), (bm + 1, bn - 1, 33, 1), (bm - 1, bn + 1, 31, 2), (2 * bm, bn, 64, 0),
                           (5, 4, 7, 3), (bm + 5, 2 * bn + 3, 257, 1), (bm, bn, 192, 0), (2 * bm + 7, bn + 9, 450, 3),
                           (4, 5, 1, 1), (bm, 2 * bn, 512, 0)]:
        check(M, N, K, ta, tb, shift, name)


@pytest.mark.parametrize("M,N,K", [(1, 1, 5000), (2, 300, 65), (3, 17, 64), (300, 1, 100), (65, 3, 1000), (1, 1, 1)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("force", [None, "128x128", "32x32"])
def test_few_rows_or_columns(M, N, K, ta, tb, force, monkeypatch):
    if force:
        monkeypatch.setenv("MX_GEMM_TILE", force)
    check(M, N, K, ta, tb, 1, "few rows")


@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
def test_empty_inner_dimension(ta, tb):
    say("product K = 0")
    A, B = torch.empty((0, 70) if ta else (70, 0), device="cuda"), torch.empty((33, 0) if tb else (0, 33), device="cuda")
    C = torch.full((70, 33), 7.0, device="cuda")
    abi.mx_map_map_reduce_f32(ta, tb, A, B, C)
    assert not C.any()


def test_special_values_stay_in_their_rows_and_columns():
    """An infinity and a NaN reach exactly the row or column of C that reads them, whatever pads the tiles."""
    for M, N, K in [(70, 50, 40), (300, 260, 200), (700, 900, 333)]:
        A, B = W.dense_f32(M, N, K, seed=5)
        A[3, K - 1], B[2, 7] = np.inf, np.nan
        C = torch.empty((M, N), device="cuda")
        abi.mx_map_map_reduce_f32(0, 0, placed(A, 0), placed(B, 0), C)
        bad = ~np.isfinite(C.cpu().numpy())
        want = np.zeros((M, N), dtype=bool)
        want[3], want[:, 7] = True, True
        assert np.array_equal(bad, want)


def test_more_threads_than_a_grid_row_holds():
    """A column of 2^27 elements and more: as many tiles of a few rows as that is are still one launch."""
    n = (1 << 27) + 37
    say("product long column", n)
    x = torch.rand(n, 1, device="cuda") * 2 - 1
    b = torch.tensor([[1.5]], device="cuda")
    for ta in (0, 1):
        C = torch.full((n, 1), 7.0, device="cuda")
        abi.mx_map_map_reduce_f32(ta, 0, x.view(1, n) if ta else x, b, C)
        assert torch.equal(C, x * 1.5)


def test_more_tiles_than_a_grid_row(monkeypatch):
    """1025 x 1025 tiles of 16 x 16: 2^20 blocks and 2049 in the second row of the grid."""
    M = N = 16400
    K = 300
    say("product two grid rows", M, N, K)
    monkeypatch.setenv("MX_GEMM_TILE", "16x16")
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B = (torch.rand(M, K, device="cuda", generator=g) * 2 - 1 for _ in range(2))
    C = torch.full((M, N), 7.0, device="cuda")
    abi.mx_map_map_reduce_f32(0, 1, A, B, C)
    for r in range(0, M, 4100):
        a, b = A[r:r + 4100].double(), B.t().contiguous().double()
        err = (C[r:r + 4100].double() - a @ b).abs()
        assert bool((err <= (K + 2) * 2.0 ** -24 * (a.abs() @ b.abs())).all())


@pytest.mark.parametrize("K", [0, 1, 31, 32, 33, 64, 65, 96, 128, 129, 160, 256, 257])
def test_waves_by_slices(K, monkeypatch):
    """Past three rounds of blocks the direct tiles take as many waves as K has slices, at most eight or four."""
    M, N = 1300, 611  # 3198 and 820 tiles
    for name in ("16x16", "32x32"):
        monkeypatch.setenv("MX_GEMM_TILE", name)
        for ta, tb in ((0, 0), (0, 1), (1, 0), (1, 1)):
            if K:
                check(M, N, K, ta, tb, 1, name)
            else:
                C = torch.full((M, N), 7.0, device="cuda")
                abi.mx_map_map_reduce_f32(ta, tb, torch.empty((0, M) if ta else (M, 0), device="cuda"),
                                          torch.empty((N, 0) if tb else (0, N), device="cuda"), C)
                assert not C.any()


def test_forced_sides_without_their_number_of_waves(monkeypatch):
    """A forced shape with a number of waves that no kernel has, or not for this product, is the shape of those sides."""
    M, N, K = 300, 200, 1000
    say("product forced sides")
    A, B = (torch.rand(*s, device="cuda") * 2 - 1 for s in ((M, K), (K, N)))

    def product(name):
        monkeypatch.setenv("MX_GEMM_TILE", name)
        C = torch.empty((M, N), device="cuda")
        abi.mx_map_map_reduce_f32(0, 0, A, B, C)
        return C

    # the shapes add K in different orders
    assert not torch.equal(product("128x64"), product("16x16")) and not torch.equal(product("128x128"), product("16x16"))
    assert torch.equal(product("128x64w8"), product("128x64"))
    for name in ("128x128w8", "128x128w8b", "128x128w16"):
        assert torch.equal(product(name), product("128x128"))
