"""The transpose kernel's launches: every pair split (9 and 10 tiles), whole pairs with
several rotation steps per iteration (12 and 17 tiles), and partly split ones with two,
three and five rows of split pairs (24, 25 and 27 tiles), for both kernels and the
periodic distance.  The workspace holds NaN bytes, so an extra slot that nothing wrote
would show; gradients against FP64 reverse-mode differentiation of the same steps,
within the adjoint's 1e-4 (norm-wise; parameters relative to the largest)."""
from ctypes import byref, c_double

import numpy as np
import pytest
import torch

from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")
from paper_2504_13379_amd import _lib as L  # noqa: E402

BETA, THETA, DT, STEPS, EVERY, TOL = 20.0, 0.2, 0.05, 3, 2, 1e-4


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


def _adjoint(ctx, prob, k, f, u0, ubar, fill):
    n = prob.n
    u = torch.from_numpy(u0.reshape(1, -1).copy()).cuda()
    ck = prob.integrate(k, f, u, DT, STEPS, ckpt_every=EVERY)
    nbytes = L.lib().nfr_adjoint_workspace_size(prob.handle, STEPS, EVERY)
    ws = torch.full((nbytes + 256,), fill, dtype=torch.uint8, device="cuda")
    ub = torch.from_numpy(ubar).cuda()
    gu = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    gp = (c_double * 5)()
    fs = f.struct(ctx.device)
    torch.cuda.synchronize()
    L.check(L.lib().nfr_adjoint(prob.handle, byref(k), byref(fs), ck.data_ptr(), EVERY, STEPS, DT, ub.data_ptr(),
                                gu.data_ptr(), gp, ws.data_ptr() + (-ws.data_ptr()) % 256, nbytes))
    torch.cuda.synchronize()
    return gu.cpu().numpy(), np.array(list(gp))


def _reference(x, q, kind, p, period, u0, ubar):
    X, Q = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    d = X[:, None, :] - X[None, :, :]
    if period:
        d[..., :2] -= period * torch.round(d[..., :2] / period)
    r2 = (d * d).sum(2)
    del d
    dist = r2 if kind == 0 else torch.sqrt(r2)
    par = torch.tensor(list(p) + [THETA], dtype=torch.float64, device="cuda", requires_grad=True)
    scale = (lambda s: s * s) if kind == 0 else (lambda s: s)
    W = par[0] * torch.exp(-dist / scale(par[1])) - par[2] * torch.exp(-dist / scale(par[3]))
    F = lambda v: W @ (Q * torch.sigmoid(BETA * (v - par[4]))) - v  # noqa: E731
    start = torch.from_numpy(u0).cuda().requires_grad_(True)
    u = start
    for _ in range(STEPS):
        k1 = F(u)
        k2 = F(u + 0.5 * DT * k1)
        k3 = F(u + 0.5 * DT * k2)
        k4 = F(u + DT * k3)
        u = u + DT / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
    u.backward(torch.from_numpy(ubar).cuda())
    return start.grad.cpu().numpy(), par.grad.cpu().numpy()


@pytest.mark.parametrize("n,kind,period", [(2200, 0, 0.0), (2560, 1, 4.0), (2900, 0, 0.0), (2900, 1, 0.0), (4352, 0, 4.0),
                                           (5900, 0, 0.0), (5900, 1, 0.0), (6400, 0, 0.0), (6400, 1, 4.0), (6700, 1, 0.0)])
def test_gradients(ctx, n, kind, period):
    rng = np.random.default_rng(n)
    x = S.fibonacci_sphere(n)
    if period:
        x[:, 2] = 0.0
    q = 4 * np.pi / n * rng.uniform(0.5, 1.1, size=n)
    u0, ubar = rng.normal(0.2, 0.4, size=n), rng.normal(size=n)
    p = (1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.33)
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), period=period)
    k, f = P.kernel_struct(kind, *p), P.Firing(BETA, THETA)
    gu, gp = _adjoint(ctx, prob, k, f, u0, ubar, 255)
    gu0, gp0 = _adjoint(ctx, prob, k, f, u0, ubar, 0)
    np.testing.assert_array_equal(gu, gu0)
    np.testing.assert_array_equal(gp, gp0)
    ru, rp = _reference(x, q, kind, p, period, u0, ubar)
    assert np.max(np.abs(gu - ru)) <= TOL * np.max(np.abs(ru))
    assert np.max(np.abs(gp - rp)) <= TOL * np.max(np.abs(rp))


@pytest.mark.parametrize("n,more", [(2560, 3072), (6400, 7168)])
@pytest.mark.parametrize("kind", [0, 1])
def test_split_pairs_give_the_same_bits(ctx, n, more, kind):
    """Two groups of 64 nodes carry all weights and cotangents, so every pair sum has
    two terms that are not 0 and its FP64 total has one value in any order.  `more`
    nodes of weight 0 behind them change the tile pairs from split to whole."""
    rng = np.random.default_rng(n)
    x = S.fibonacci_sphere(more)
    x = x[rng.permutation(more)]
    q, ubar = np.zeros(more), np.zeros(more)
    both = np.concatenate([np.arange(5 * 256 + 64, 5 * 256 + 128), np.arange(n - 128, n - 64)])
    q[both] = 0.05 * rng.uniform(0.5, 1.0, size=128)
    ubar[both] = rng.normal(size=128)
    u0 = rng.normal(0.2, 0.4, size=more)
    p = (1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.33)
    k, f = P.kernel_struct(kind, *p), P.Firing(BETA, THETA)
    got = []
    for m in (n, more):
        prob = P.Problem(ctx, torch.from_numpy(x[:m]).cuda(), torch.from_numpy(q[:m]).cuda())
        got.append(_adjoint(ctx, prob, k, f, u0[:m], ubar[:m], 255)[0][:n])
    assert np.any(got[0][both] != ubar[both])
    np.testing.assert_array_equal(got[0], got[1])
