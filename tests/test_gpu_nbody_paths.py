"""The schedules of the N-body pair sum (direct, symmetric, sliced) at the edges of their ranges, in both directions,
against the binary64 formulas on sampled bodies; calls in place; and a reverse sweep run twice from one forward."""
import numpy as np
import pytest
import torch

import workloads as W
from parity import say

import paper_2211_00621_amd as mx  # noqa: E402
from test_gpu_nbody import DT, EPS2, G, accel_magnitude, check_bodies, to4, v4, vjp_magnitude

pytestmark = pytest.mark.gpu
abi, api = mx.abi, mx.api


def exact(pos, m, abar, rows):
    """Acceleration and transposed-Jacobian product of the bodies `rows` in binary64."""
    x, mm, ab = (torch.from_numpy(t).to("cuda").double() for t in (pos, m, abar))
    a, v = torch.empty(len(rows), 3, device="cuda", dtype=torch.float64), torch.empty(
        len(rows), 3, device="cuda", dtype=torch.float64)
    for p in range(0, len(rows), 64):
        r = torch.from_numpy(rows[p:p + 64]).to("cuda")
        d = x[None] - x[r][:, None]
        s = (d * d).sum(-1) + float(np.float32(EPS2))
        phi = s ** -1.5
        a[p:p + 64] = G * ((mm[None] * phi)[..., None] * d).sum(1)
        w = mm[r][:, None, None] * ab[None] - mm[None, :, None] * ab[r][:, None]
        v[p:p + 64] = G * (phi[..., None] * w - (3 * phi / s * (d * w).sum(-1))[..., None] * d).sum(1)
    return a.cpu().numpy(), v.cpu().numpy()


# direct up to 4096 bodies (four per block up to 1024, then eight), symmetric up to 65 536 (sets of 256), then sliced
@pytest.mark.parametrize("n", [3, 63, 65, 1023, 1024, 1025, 1031, 4095, 4096, 4097, 4352, 4353, 8191, 20000, 65536,
                               65537])
def test_pair_schedules_vs_binary64(n):
    say("nbody schedules", n)
    pos, m, _ = W.nbody(n, seed=n)
    abar = np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(min(n, 8)), np.arange(max(0, n - 8), n),
                                     np.random.default_rng(1).integers(0, n, 240)]))
    p4, a4 = torch.from_numpy(to4(pos, m)).to("cuda"), torch.from_numpy(v4(abar)).to("cuda")
    ws = torch.zeros(abi.mx_nbody_pair_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    acc, out = torch.empty_like(p4), torch.empty_like(p4)
    abi.mx_nbody_accel_f32(p4, EPS2, G, acc, ws)
    abi.mx_nbody_accel_vjp_f32(p4, a4, EPS2, G, out, ws)
    ra, rv = exact(pos, m, abar, rows)
    check_bodies(acc.cpu().numpy()[rows, :3], ra, accel_magnitude(pos, m, EPS2, rows=rows, chunk=16), n, what="a")
    check_bodies(out.cpu().numpy()[rows, :3], rv, vjp_magnitude(pos, m, abar, EPS2, rows=rows, chunk=16), n,
                 what="vjp")
    again = torch.empty_like(p4)
    abi.mx_nbody_accel_vjp_f32(p4, a4, EPS2, G, again, ws)
    assert torch.equal(again, out)
    # one step and one reverse step apply the same sums
    xo, vo, xb, vb = (torch.empty_like(p4) for _ in range(4))
    abi.mx_nbody_step_f32(p4, a4, EPS2, G, DT, xo, vo, ws)
    abi.mx_nbody_adjoint_step_f32(p4, p4, a4, EPS2, G, DT, xb, vb, ws)
    assert torch.allclose(vo[:, :3], a4[:, :3] + DT * acc[:, :3], rtol=1e-6, atol=1e-6)
    assert torch.allclose(xb[:, :3], p4[:, :3] + DT * out[:, :3], rtol=1e-6, atol=1e-6)
    assert torch.equal(xo[:, 3], p4[:, 3])


@pytest.mark.parametrize("n", [200, 1000, 5000])
def test_in_place_outputs(n):
    """The acceleration written over the positions and the product over its adjoint give the same sums."""
    say("nbody in place", n)
    pos, m, _ = W.nbody(n, seed=n)
    p4 = torch.from_numpy(to4(pos, m)).to("cuda")
    a4 = torch.randn(n, 4, device="cuda")
    a4[:, 3] = 0
    ws = torch.zeros(abi.mx_nbody_pair_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    acc, out, p, a = torch.empty_like(p4), torch.empty_like(p4), p4.clone(), a4.clone()
    abi.mx_nbody_accel_f32(p4, EPS2, G, acc, ws)
    abi.mx_nbody_accel_f32(p, EPS2, G, p, ws)
    abi.mx_nbody_accel_vjp_f32(p4, a4, EPS2, G, out, ws)
    abi.mx_nbody_accel_vjp_f32(p4, a, EPS2, G, a, ws)
    S, T = accel_magnitude(pos, m, EPS2), vjp_magnitude(pos, m, a4[:, :3].cpu().numpy(), EPS2)
    check_bodies(p.cpu().numpy()[:, :3], acc.cpu().numpy()[:, :3].astype(np.float64), S, n, what="a in place")
    check_bodies(a.cpu().numpy()[:, :3], out.cpu().numpy()[:, :3].astype(np.float64), T, n, what="vjp in place")


@pytest.mark.parametrize("steps,ckpt", [(1, 1), (7, 3), (6, 3), (5, 9)])
def test_reverse_sweep_twice_from_one_forward(steps, ckpt):
    """The reverse sweep leaves what the forward stored intact, so it can run again, and equals the fused call."""
    n = 300
    say("nbody reverse twice", steps, ckpt)
    pos, m, vel = W.nbody(n, seed=9)
    p4, v = torch.from_numpy(to4(pos, m)).to("cuda"), torch.from_numpy(v4(vel)).to("cuda")
    ke, gx, gv = api.nbody_ke_grad(p4, v, EPS2, G, DT, steps, ckpt)
    ws = torch.zeros(abi.mx_nbody_workspace_bytes(n, steps, ckpt), dtype=torch.uint8, device="cuda")
    ke2 = torch.empty((), device="cuda")
    abi.mx_nbody_ke_f32(p4, v, EPS2, G, DT, steps, ckpt, ke2, ws)
    assert torch.equal(ke, ke2)
    for _ in range(2):
        hx, hv = torch.full_like(p4, 7.0), torch.full_like(p4, 7.0)
        abi.mx_nbody_ke_vjp_f32(p4, v, EPS2, G, DT, steps, ckpt, None, hx, hv, ws)
        assert torch.equal(hx, gx) and torch.equal(hv, gv)


@pytest.mark.parametrize("n", [200, 1000, 4096])
@pytest.mark.parametrize("over", ["pos4", "vel4"])
def test_gradients_over_the_state(n, over):
    """A gradient of the loop, or the velocities' adjoint of a step, written over the state that the sweep reads."""
    say("nbody gradients over the state", n, over)
    pos, m, vel = W.nbody(n, seed=n)
    p4, v = torch.from_numpy(to4(pos, m)).to("cuda"), torch.from_numpy(v4(vel)).to("cuda")
    eps2, steps, ckpt = 0.05 ** 2, 3, 2
    ke, gx, gv = api.nbody_ke_grad(p4, v, eps2, G, DT, steps, ckpt)
    ws = torch.zeros(abi.mx_nbody_workspace_bytes(n, steps, ckpt), dtype=torch.uint8, device="cuda")
    S = float(torch.cat([gx, gv]).abs().max())
    for which in ("gx4", "gv4"):
        s = {"pos4": p4.clone(), "vel4": v.clone(), "other": torch.empty_like(p4)}
        gx2, gv2 = (s[over], s["other"]) if which == "gx4" else (s["other"], s[over])
        ke2 = torch.empty((), device="cuda")
        abi.mx_nbody_ke_grad_f32(s["pos4"], s["vel4"], eps2, G, DT, steps, ckpt, ke2, gx2, gv2, ws)
        # the schedules' sums differ by their rounding alone
        assert torch.equal(ke2, ke)
        assert float((gx2 - gx).abs().max()) <= 1e-4 * S and float((gv2 - gv).abs().max()) <= 1e-4 * S, which
    xb, vb, wp = torch.randn_like(p4), torch.randn_like(p4), torch.zeros(
        abi.mx_nbody_pair_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    xo, vo, x2, p2 = torch.empty_like(p4), torch.empty_like(p4), torch.empty_like(p4), p4.clone()
    abi.mx_nbody_adjoint_step_f32(p4, xb, vb, eps2, G, DT, xo, vo, wp)
    abi.mx_nbody_adjoint_step_f32(p2, xb, vb, eps2, G, DT, x2, p2, wp)
    assert torch.equal(p2, vo)
    assert float((x2 - xo).abs().max()) <= 1e-4 * float((xo - xb).abs().max())
