"""One state on the symmetric kernel where the last tile pairs are split into their
source groups: tile counts with the split pairs in one row of the order (32, 45
tiles), in two (40) and none (28), padded and exact node counts, both kernels and
the periodic distance.  The workspace holds NaN bytes, so an extra slot that nothing
wrote would show; one Euler-like step of RK4 against the FP64 operator."""
import numpy as np
import pytest
import torch

from oracle import neural_field as NF
from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


@pytest.mark.parametrize("n,kind,period", [(7168, 0, 0.0), (8192, 0, 0.0), (7937, 1, 0.0), (10007, 0, 0.0),
                                           (11300, 1, 0.0), (10240, 0, 4.0)])
def test_split_pairs(ctx, n, kind, period):
    rng = np.random.default_rng(n)
    x = S.fibonacci_sphere(n)
    if period:
        x[:, 2] = 0.0
    q = 4 * np.pi / n * rng.uniform(-0.2, 1.1, size=n)
    u0 = rng.normal(0.2, 0.4, size=n)
    p = (1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.3)
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), period=period)
    k, f, dt = P.kernel_struct(kind, *p), P.Firing(20.0, 0.2), 0.05
    runs = []
    for fill in (255, 0):
        u = torch.from_numpy(u0.reshape(1, -1).copy()).cuda()
        ws = prob.integrate_workspace(1, P.FORM_ONTHEFLY_FP32)
        ws.fill_(fill)
        torch.cuda.synchronize()
        prob.integrate(k, f, u, dt, 1, ws=ws)
        ctx.stream.synchronize()
        runs.append(u.cpu().numpy()[0])
    np.testing.assert_array_equal(runs[0], runs[1])
    # the same step in FP64 on the GPU (plain torch)
    X, Q, v0 = (torch.from_numpy(a).cuda() for a in (x, q, u0))
    W = torch.empty((n, n), dtype=torch.float64, device="cuda")
    for r in range(0, n, 1024):
        r2 = 0.0
        for d in range(3):
            c = X[r:r + 1024, d, None] - X[None, :, d]
            if period and d < 2:
                c = c - period * torch.round(c / period)
            r2 = r2 + c * c
        e = (lambda s: torch.exp(-r2 / s ** 2)) if kind == 0 else (lambda s: torch.exp(-torch.sqrt(r2) / s))
        W[r:r + 1024] = p[0] * e(p[1]) - p[2] * e(p[3])
    F = lambda v: W @ (Q / (1.0 + torch.exp(-20.0 * (v - 0.2)))) - v  # noqa: E731
    k1 = F(v0)
    k2 = F(v0 + 0.5 * dt * k1)
    k3 = F(v0 + 0.5 * dt * k2)
    k4 = F(v0 + dt * k3)
    ref = (v0 + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)).cpu().numpy()
    # FP32 pair sums: 1e-5 of sum |w g| (a few units here) times dt
    assert float(NF.rel_linf(runs[0], ref).max()) <= 1e-6
