"""The split of the multi-state on-the-fly FP32 sum into slots.  Its partial sums take
at most 256 MB (or one slot), and from one padded size to the next the workspace grows
less than the 4 times that a split bounded for nfr_apply_noalloc alone jumped by.  And
nfr_apply_noalloc takes the applications it always took where nfr_apply's workspace
exceeds its scratch, in groups of states, the last of them a single state, with the
same bits; what it refused it refuses."""
import math

import numpy as np
import pytest
import torch

from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")
from paper_2504_13379_amd import _lib as L  # noqa: E402

FORM = L.FORM_ONTHEFLY_FP32


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


def test_workspace_does_not_jump(ctx):
    x = torch.rand((65536, 3), dtype=torch.float64, device="cuda")
    q = torch.rand(65536, dtype=torch.float64, device="cuda")
    states = (2, 8, 16, 24, 40, 64, 113)
    last = None
    for n in range(4096, 65537, 256):
        prob = P.Problem(ctx, x[:n], q[:n])
        need = [L.lib().nfr_apply_workspace_size(prob.handle, B, FORM) for B in states]
        for B, a, b in zip(states, last or need, need):
            assert max(a / b, b / a) <= 3.6, (n, B, a, b)
            assert b <= 4 * n * B + max(256 << 20, 8 * n * B), (n, B, b)
        last = need


def _case(ctx, n, B):
    rng = np.random.default_rng(n)
    x = torch.from_numpy(S.fibonacci_sphere(n)).cuda()
    prob = P.Problem(ctx, x, torch.from_numpy(4 * math.pi / n * rng.uniform(0.9, 1.1, n)).cuda())
    u = torch.from_numpy(rng.normal(0.2, 0.3, size=(B, n))).cuda()
    return prob, P.kernel_struct(0, 1.0, 0.15, 0.5, 0.4), P.Firing(20.0, torch.from_numpy(rng.uniform(0.15, 0.3, B)).cuda()), u


@pytest.mark.parametrize("n,B", [(33000, 50), (22000, 9), (600000, 4)])
def test_noalloc_in_groups_equals_apply(ctx, n, B):
    prob, k, f, u = _case(ctx, n, B)
    assert L.lib().nfr_apply_workspace_size(prob.handle, B, FORM) > L.NFR_APPLY_NOALLOC_MAX_BYTES
    ref = prob.apply(k, f, u, form=FORM)
    out = torch.full_like(u, float("nan"))
    prob.apply_noalloc(k, f, u, out, form=FORM)
    ctx.stream.synchronize()
    assert bool(torch.isfinite(ref).all())
    assert torch.equal(ref, out)


@pytest.mark.parametrize("n,B", [(65536, 64), (33000, 64)])
def test_noalloc_refuses_as_before(ctx, n, B):
    prob, k, f, u = _case(ctx, n, B)
    out = torch.zeros_like(u)
    with pytest.raises(P.NfrError) as e:
        prob.apply_noalloc(k, f, u, out, form=FORM)
    assert e.value.status == L.NFR_ERR_WORKSPACE
    ctx.stream.synchronize()
    assert float(out.abs().max()) == 0.0
