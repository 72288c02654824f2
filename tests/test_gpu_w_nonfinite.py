"""Entries of the precomputed W at coordinates that are not finite, in every W form:
0 in a column of weight 0 (and in the padding), NaN where the distance is NaN, 0 at an
infinite distance, finite everywhere else; so a node kept far away at infinity with
weight 0 adds nothing, and its own value is the finite sum 0.  Against FP64 NumPy."""
import numpy as np
import pytest
import torch

import paper_2504_13379_amd as P

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


@pytest.mark.parametrize("form", [P.FORM_W_FP32, P.FORM_W_BF16X3, P.FORM_W_FP16X3])
@pytest.mark.parametrize("kind,kern", [(0, (1.0, 0.15, 0.5, 0.4)), (1, (2.0, 0.1, 1.0, 0.3))])
def test_entries(ctx, form, kind, kern):
    n = 300
    rng = np.random.default_rng(kind)
    x = rng.uniform(-1.0, 1.0, size=(n, 3))
    q = rng.uniform(0.2, 1.0, size=n) / n
    q[[5, 40, 41]] = 0.0
    x[40], x[41], x[170, 1], x[290, 2] = INF, (NAN, 0.0, 0.0), -INF, NAN      # 40 and 41 of weight 0
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda())
    k = P.kernel_struct(kind, *kern)
    with np.errstate(invalid="ignore"):
        r2 = ((x[:, None] - x[None]) ** 2).sum(2)
        e = (lambda s: np.exp(-r2 / s ** 2)) if kind == 0 else (lambda s: np.exp(-np.sqrt(r2) / s))
        ref = np.where(q[None] == 0.0, 0.0, (kern[0] * e(kern[1]) - kern[2] * e(kern[3])) * q[None])
    npad = prob.npad
    W = prob.w_build(k, form)
    ctx.stream.synchronize()
    if form == P.FORM_W_FP32:
        got = W.view(torch.float32)[:n * npad].reshape(n, npad).cpu().numpy().astype(np.float64)
        assert not np.signbit(got[:, q_pad(q, npad) == 0.0]).any()
    else:
        dt, c = (torch.bfloat16, 0) if form == P.FORM_W_BF16X3 else (torch.float16, 11)
        sw = float(W[:4].view(torch.float32)[0])
        t = W[256:256 + 4 * npad * npad].view(dt).to(torch.float64).cpu().numpy()
        t = t.reshape(npad // 128, npad // 16, 2, 4, 2, 32, 8).transpose(2, 0, 3, 5, 1, 4, 6).reshape(2, npad, npad)
        got = ((t[0] + 2.0 ** -c * t[1]) * 2.0 ** -sw)[:n]
    assert np.all(got[:, n:] == 0.0)
    np.testing.assert_array_equal(np.isnan(got[:, :n]), np.isnan(ref))
    ok = ~np.isnan(ref)
    # 16 bits (BF16) of each entry, and FP64 rounding of the cancelling terms
    assert np.max(np.abs(got[:, :n] - ref)[ok]) <= 2.0 ** -16 * np.max(np.abs(ref[ok]))
    assert np.all(got[40, ok[40].nonzero()[0]] == 0.0)


def q_pad(q, npad):
    return np.concatenate([q, np.zeros(npad - len(q))])


@pytest.mark.parametrize("form", [P.FORM_W_FP32, P.FORM_W_BF16X3, P.FORM_W_FP16X3])
def test_weightless_node_at_infinity(ctx, form):
    n = 700
    rng = np.random.default_rng(4)
    x = rng.uniform(-1.0, 1.0, size=(n, 3))
    q = rng.uniform(0.2, 1.0, size=n) / n
    u = torch.from_numpy(rng.normal(0.2, 0.4, size=(3, n))).cuda()
    k, f = P.kernel_struct(0, 1.0, 0.15, 0.5, 0.4), P.Firing(20.0, 0.2)
    q[123] = 0.0
    out = []
    for far in (x[123].copy(), (INF, 0.0, 0.0)):
        x[123] = far
        prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda())
        y = prob.apply(k, f, u, form=form, W=prob.w_build(k, form))
        ctx.stream.synchronize()
        out.append(y.cpu().numpy())
    rest = np.arange(n) != 123
    np.testing.assert_array_equal(out[1][:, rest], out[0][:, rest])
    assert np.all(out[1][:, 123] == 0.0)
