"""The vector-unit multi-state sum (2 to 8 states) where its plan changes the
targets per lane, and where a chunk gives some waves of a workgroup no source tile:
256 to a few thousand nodes, against the FP64 oracle (1e-5 of sum |w g|), and each
state the same within FP64 rounding in calls of other state counts (the FP32 sums
of 256 sources are the same)."""
import math

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


@pytest.mark.parametrize("n", [200, 257, 1025, 2900, 5100])
@pytest.mark.parametrize("kind", [0, 1])
def test_plans_agree(ctx, n, kind):
    rng = np.random.default_rng(n)
    x = S.fibonacci_sphere(n)
    q = np.full(n, 4 * math.pi / n) * rng.uniform(-0.2, 1.1, size=n)
    U = rng.normal(0.2, 0.4, size=(8, n))
    theta = rng.uniform(0.1, 0.3, size=8)
    p = (1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.33)
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda())
    k = P.kernel_struct(kind, *p)
    G = q[None, :] * NF.firing(U, 20.0, theta)
    w = NF.kernel_matrix(x, kind, p)
    scale = np.abs(G) @ np.abs(w).T
    ref = G @ w.T
    first = None
    for B in (8, 2, 3, 4, 5):
        y = prob.apply(k, P.Firing(20.0, torch.from_numpy(theta[:B]).cuda()), torch.from_numpy(U[:B].copy()).cuda())
        ctx.stream.synchronize()
        y = y.cpu().numpy()
        assert np.max(np.abs(y - ref[:B]) / scale[:B]) <= 1e-5
        first = y if first is None else first
        assert np.max(np.abs(y - first[:B]) / scale[:B]) <= 2.0 ** -46
