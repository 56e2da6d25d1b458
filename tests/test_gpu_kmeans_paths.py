"""The k-means step at every remainder of the dimension modulo four, on both sides of its paddings (d 32 / 33 / 64, k 16 /
17, 32 / 33, 64 / 65), with and without copies of the sums, unaligned X, partial last chunks, one label for all points;
and the SSE with its gradient in chunks of one and two vectors per thread.  Labels and counts are exact, the centroids
within the rounding of the means (a chunk's points are added in float32 to at most 64 sums in a row per wave)."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import say

import paper_2211_00621_amd as mx  # noqa: E402

pytestmark = pytest.mark.gpu
abi = mx.abi
U = 2.0 ** -24


def slice_of(x, shift):
    t = torch.zeros(x.size + shift, device="cuda")
    t[shift:] = torch.from_numpy(x.ravel())
    return t[shift:].view(x.shape)


def blobs(n, d, k, seed, one_label=False):
    rng = np.random.default_rng(seed)
    C = rng.uniform(-1, 1, (k, d)).astype(np.float32)
    lab = np.zeros(n, np.int64) if one_label else rng.integers(0, k, n)
    return (C[lab] + 0.15 * rng.standard_normal((n, d))).astype(np.float32), C


def step(X, C, shift):
    n, d = X.shape
    k = len(C)
    ws = torch.zeros(abi.mx_kmeans_workspace_bytes(n, d, k), dtype=torch.uint8, device="cuda")
    lab = torch.full((n + 3,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(k, dtype=torch.int64, device="cuda")
    Cn = torch.zeros(k, d, device="cuda")
    abi.mx_kmeans_step_f32(slice_of(X, shift), torch.from_numpy(C).cuda(), lab[:n], cnt, Cn, ws)
    torch.cuda.synchronize()
    assert np.all(lab[n:].cpu().numpy() == -7)
    return lab[:n].cpu().numpy(), cnt.cpu().numpy(), Cn.cpu().numpy()


def check(X, C, shift):
    lab, cnt, Cn = step(X, C, shift)
    ref = O.kmeans_assign(X, C)
    assert np.array_equal(lab, ref), (X.shape, len(C), int((lab != ref).sum()))
    ref_cnt, _, ref_C = O.kmeans_update(X, ref, C)
    assert np.array_equal(cnt, ref_cnt)
    mean_abs = np.zeros(C.shape)
    np.add.at(mean_abs, ref, np.abs(X.astype(np.float64)))
    mean_abs /= np.maximum(ref_cnt, 1)[:, None]
    # every sum is a chain of at most n float32 additions
    bound = (np.minimum(ref_cnt, 4096)[:, None] + 2) * U * mean_abs + U * np.abs(ref_C) + 1e-30
    assert np.all(np.abs(Cn - ref_C) <= bound), (X.shape, len(C))


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 8, 15, 16, 18, 31, 32, 33, 34, 35, 48, 50, 63, 64])
def test_dimensions(d, shift):
    say("kmeans dimension", d, shift)
    for n, k in ((1, 1), (65, 3), (4133, 10), (3000, 40)):
        check(*blobs(n, d, k, n + d), shift)


@pytest.mark.parametrize("k", [1, 2, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127])
def test_centroids(k):
    say("kmeans centroids", k)
    for n, d in ((63, 32), (5003, 32), (5003, 20), (2000, 31)):
        check(*blobs(n, d, k, k + d), 0)
    if k <= 64:
        check(*blobs(1999, 64, k, k), 0)
        check(*blobs(1999, 61, k, k), 0)


@pytest.mark.parametrize("d,k", [(8, 10), (32, 10), (32, 64), (64, 20)])
def test_one_label(d, k):
    """Every point of a chunk in one cluster: the most passes there are."""
    say("kmeans one label", d, k)
    X, C = blobs(3333, d, k, 5, one_label=True)
    check(X, C, 0)


@pytest.mark.parametrize("n,d", [(1, 1), (3, 5), (1000, 1), (700, 7), (4096, 32), (40000, 25), (40000, 26), (70000, 16),
                                 (300000, 4), (20000, 70), (3, 40000), (40, 70001)])
@pytest.mark.parametrize("shift", [0, 1])
def test_sse_and_gradient(n, d, shift):
    say("kmeans sse", n, d, shift)
    rng = np.random.default_rng(n + d)
    k = 9
    X, C = rng.uniform(-1, 1, (n, d)).astype(np.float32), rng.uniform(-1, 1, (k, d)).astype(np.float32)
    lab = rng.integers(0, k, n).astype(np.int32)
    dX, dC, dl = slice_of(X, shift), slice_of(C, shift), torch.from_numpy(lab).cuda()
    ws = torch.zeros(256 + 4096, dtype=torch.uint8, device="cuda")
    sse = torch.zeros(1, device="cuda")
    abi.mx_kmeans_sse_f32(dX, dC, dl, sse, ws)
    diff = X.astype(np.float64) - C[lab].astype(np.float64)
    ref = (diff ** 2).sum()
    # a square carries three roundings; a thread adds at most n d / 512 of them, then the trees
    assert abs(float(sse.cpu()[0]) - ref) <= (n * d / 512 + 32) * U * ref
    big = torch.full((n * d + shift + 5,), 7.0, device="cuda")
    g = torch.tensor([0.75], device="cuda")
    abi.mx_kmeans_sse_grad_f32(dX, dC, dl, g, big[shift:shift + n * d].view(n, d))
    h = big.cpu().numpy()
    assert np.all(h[:shift] == 7) and np.all(h[shift + n * d:] == 7)
    assert np.array_equal(h[shift:shift + n * d].reshape(n, d), np.float32(1.5) * (X - C[lab]))


def test_gradient_past_the_cache():
    """More than 256 MiB of X and gradient."""
    n, d, k = 1100003, 32, 8
    say("kmeans gradient past the cache", n, d)
    rng = np.random.default_rng(3)
    X, C = rng.uniform(-1, 1, (n, d)).astype(np.float32), rng.uniform(-1, 1, (k, d)).astype(np.float32)
    lab = rng.integers(0, k, n).astype(np.int32)
    G = torch.full((n, d), 7.0, device="cuda")
    abi.mx_kmeans_sse_grad_f32(torch.from_numpy(X).cuda(), torch.from_numpy(C).cuda(), torch.from_numpy(lab).cuda(),
                               torch.tensor([0.5], device="cuda"), G)
    assert np.array_equal(G.cpu().numpy(), X - C[lab])


@pytest.mark.parametrize("n,d", [(683, 3), (682, 3), (1024, 2), (1025, 2), (2047, 1), (2049, 1), (512, 4), (513, 4), (257, 8),
                                 (87381, 3), (87382, 3), (262144, 1), (262145, 1), (131072, 4), (131073, 4), (262143, 2),
                                 (262145, 2)])
def test_small_sse_edges(n, d):
    """Sums of one block (2048 elements), an element per thread (2^18) and a vector (2^19), and the first past each."""
    test_sse_and_gradient(n, d, 1)


@pytest.mark.parametrize("n,d", [(43690, 3), (43691, 3), (65536, 2), (131073, 1), (74898, 7), (74899, 7), (131072, 4),
                                 (524289, 1), (349525, 3), (349526, 3), (16384, 32), (1048577, 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_sse_last_of_the_small_passes(n, d, shift):
    """Sums of 2^17 and 2^19 elements and gradients of 2^19 and 2^20, the last that small passes take, and the next ones."""
    test_sse_and_gradient(n, d, shift)


@pytest.mark.parametrize("n,d", [(262144, 4), (262145, 4), (131072, 8), (209715, 5), (1500003, 1), (1048580, 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_sse_last_vectors_of_the_small_passes_and_labels_by_four(n, d, shift):
    """Sums and gradients of 2^20 elements by vectors and the next ones; points of one dimension in larger passes."""
    test_sse_and_gradient(n, d, shift)
