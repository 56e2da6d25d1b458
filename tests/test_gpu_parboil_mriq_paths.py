"""mri-q at the edges of its work splits (voxels per lane, waves per block), of its tiles of samples and of the range in
which the hardware reduces the angle, within the bound of the parity test."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import say

import paper_2211_00621_amd as mx  # noqa: E402
from test_gpu_parboil import dev, host, mriq_bound, mriq_inputs

pytestmark = pytest.mark.gpu
abi = mx.abi


def run(k, phi, x):
    nv = len(x[0])
    qr, qi = (torch.full((nv,), 7.0, device="cuda") for _ in range(2))
    abi.mx_mriq_f32(*[dev(a) for a in k], dev(phi), *[dev(a) for a in x], qr, qi)
    return host(qr), host(qi)


# one voxel per lane up to 2^15 voxels, two below 3 2^16, four from there; tiles of 1024 samples, by fours
@pytest.mark.parametrize("nv", [63, 65, (1 << 15) - 1, (1 << 15) + 1, (3 << 16) - 1, 3 << 16, (3 << 16) + 257])
@pytest.mark.parametrize("nk", [0, 3, 61, 1023, 1029])
@pytest.mark.parametrize("scale", [1.0, 40.0])
def test_mriq_splits(nv, nk, scale):
    say("mriq splits", nv, nk, scale)
    k, phi, x = mriq_inputs(nk, nv, nk + nv)
    k = [np.float32(scale) * c for c in k]  # 40: angles past 250 revolutions in some lanes
    qr, qi = run(k, phi, x)
    if nk == 0:
        assert not qr.any() and not qi.any()
        return
    idx = np.unique(np.concatenate([np.arange(min(nv, 64)), np.random.default_rng(2).integers(0, nv, 64),
                                    np.arange(nv - min(nv, 300), nv)]))
    rr, ri = O.mriq(*k, phi, *[xc[idx] for xc in x])
    b = mriq_bound(k, phi, x, idx)
    assert np.all(np.abs(qr[idx] - rr) <= b) and np.all(np.abs(qi[idx] - ri) <= b)


def test_mriq_large_angle_in_one_tile():
    """A tile with one far sample reduces its angles, its neighbours do not; non-finite voxels stay their own."""
    nk, nv = 2100, 5000
    say("mriq large angle")
    k, phi, x = mriq_inputs(nk, nv, 3)
    k[1][1500] = np.float32(3e6)
    x[0][17], x[2][2000] = np.inf, np.nan
    qr, qi = run(k, phi, x)
    ok = np.ones(nv, dtype=bool)
    ok[[17, 2000]] = False
    assert np.isnan(qr[~ok]).all() and np.isnan(qi[~ok]).all()
    idx = np.flatnonzero(ok)[:1500]
    rr, ri = O.mriq(*k, phi, *[xc[idx] for xc in x])
    b = mriq_bound(k, phi, x, idx)
    assert np.all(np.abs(qr[idx] - rr) <= b) and np.all(np.abs(qi[idx] - ri) <= b)


@pytest.mark.parametrize("nv", [1, 511, 513, (1 << 19) - 1, 1 << 19])
@pytest.mark.parametrize("nk", [1, 4, 16, 17, 40, 41])
def test_mriq_few_samples(nv, nk):
    """Too few samples for the waves of a block to share: a wave for each two voxels of its lanes."""
    test_mriq_splits(nv, nk, 1.0)
    test_mriq_splits(nv, nk, 40.0)


@pytest.mark.parametrize("nk,nv", [(1, 1000), (2, 513), (3, 513), (2, 200001), (100, 3 << 16), (101, 3 << 16), (100, (3 << 16) - 1)])
def test_mriq_samples_singly_and_by_wave(nk, nv):
    """One or two samples without padding to four, and the most that a wave takes alone where the voxels fill the chip."""
    test_mriq_splits(nv, nk, 1.0)
    test_mriq_splits(nv, nk, 40.0)
