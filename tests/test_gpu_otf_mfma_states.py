"""The multi-state on-the-fly FP32 sum with its products on the matrix cores: the
state counts at which the number of 16-state groups and of state blocks changes,
padded and exact node counts.  Every state's sums are the vector form's bit for bit,
so a state gives the same result within FP64 rounding (the FP64 slots are split
differently) alone in an 8-state call and beside others; and each stays within the
on-the-fly tolerance of the FP64 oracle."""
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


@pytest.mark.parametrize("B", [9, 16, 17, 33, 49, 64, 65, 97])
@pytest.mark.parametrize("n,kind,period", [(255, 0, 0.0), (1537, 1, 0.0), (700, 0, 4.0)])
def test_states_match_vector_form_and_oracle(ctx, B, n, kind, period):
    rng = np.random.default_rng(B + n)
    x = S.fibonacci_sphere(n)
    if period:
        x[:, 2] = 0.0
    q = np.full(n, 4 * math.pi / n) * rng.uniform(-0.2, 1.1, size=n)
    U = rng.normal(0.2, 0.4, size=(B, n))
    theta = rng.uniform(0.1, 0.3, size=B)
    p = (1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.33)
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), period=period)
    k = P.kernel_struct(kind, *p)
    y = prob.apply(k, P.Firing(20.0, torch.from_numpy(theta).cuda()), torch.from_numpy(U).cuda(),
                   form=P.FORM_ONTHEFLY_FP32)
    parts = [prob.apply(k, P.Firing(20.0, torch.from_numpy(theta[b:b + 8]).cuda()), torch.from_numpy(U[b:b + 8]).cuda(),
                        form=P.FORM_ONTHEFLY_FP32) for b in range(0, B, 8) if B - b >= 8]
    ctx.stream.synchronize()
    y = y.cpu().numpy()
    v = torch.cat(parts).cpu().numpy()
    G = q[None, :] * NF.firing(U, 20.0, theta)
    w = NF.kernel_matrix(x, kind, p, period=period) if period else NF.kernel_matrix(x, kind, p)
    scale = np.abs(G) @ np.abs(w).T
    # FP64 sums of a few hundred 256-source totals, in another order
    assert np.max(np.abs(y[:len(v)] - v) / scale[:len(v)]) <= 2.0 ** -46
    assert np.max(np.abs(y - G @ w.T) / scale) <= 1e-5
