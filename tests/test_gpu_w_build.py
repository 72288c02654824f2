"""Entries of the precomputed W against FP64 NumPy: W_FP32 rounds once to FP32
(2^-24 relative, and the FP32 subnormal grid 2^-149), the split forms keep hi + lo
of 8 + 8 (BF16) or 11 + 11 (FP16, lifted by 2^sW, remainders by 2^11) bits.  Sizes
around the row blocks of 32, the row groups of 128 and their groups of four; a
kernel so narrow that far entries underflow; the periodic distance."""
import numpy as np
import pytest
import torch

import paper_2504_13379_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


def _w64(x, q, kind, kern, period):
    d = x[:, None, :] - x[None, :, :]
    if period:
        d[..., :2] = np.abs(d[..., :2])
        d[..., :2] = np.minimum(d[..., :2], period - d[..., :2])
    r2 = (d ** 2).sum(2)
    a_e, s_e, a_i, s_i = kern
    e = (lambda s: np.exp(-r2 / s ** 2)) if kind == 0 else (lambda s: np.exp(-np.sqrt(r2) / s))
    scale = (abs(a_e) * e(s_e) + abs(a_i) * e(s_i)) * np.abs(q)[None, :]
    return (a_e * e(s_e) - a_i * e(s_i)) * q[None, :], scale


@pytest.mark.parametrize("n", [1, 31, 33, 257, 700])
@pytest.mark.parametrize("kind,kern,period", [(0, (1.0, 0.15, 0.5, 0.4), 0.0), (1, (2.0, 0.1, 1.0, 0.3), 0.0),
                                              (0, (3.0, 0.01, 0.5, 0.04), 0.0), (0, (1.0, 0.6, 0.5, 1.2), 6.0)])
def test_w_entries(ctx, n, kind, kern, period):
    rng = np.random.default_rng(n)
    x = rng.uniform(-1.5, 1.5, size=(n, 3))
    if period:
        x *= 2.0 * np.array([1.0, 1.0, 0.0])
    q = rng.uniform(-0.2, 1.0, size=n) / n
    q[n // 2] = 0.0 if n > 1 else q[0]
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), period=period)
    k = P.kernel_struct(kind, *kern)
    ref, scale = _w64(x, q, kind, kern, period)
    npad = prob.npad
    fp64 = 2.0 ** -44 * scale            # FP64 arguments up to a few hundred, cancellation of the two terms
    W = prob.w_build(k, P.FORM_W_FP32)
    ctx.stream.synchronize()
    got = W.view(torch.float32)[:n * npad].reshape(n, npad).cpu().numpy().astype(np.float64)
    assert np.all(got[:, n:] == 0.0)
    assert np.all(np.abs(got[:, :n] - ref) <= 2.0 ** -24 * np.abs(ref) + 2.0 ** -149 + fp64)
    for form, dt, bits, c in ((P.FORM_W_BF16X3, torch.bfloat16, 8, 0), (P.FORM_W_FP16X3, torch.float16, 11, 11)):
        W = prob.w_build(k, form)
        ctx.stream.synchronize()
        sw = float(W[:4].view(torch.float32)[0])
        t = W[256:256 + 4 * npad * npad].view(dt).to(torch.float64).cpu().numpy()
        t = t.reshape(npad // 128, npad // 16, 2, 4, 2, 32, 8)      # group, column block, hi/lo, row block, h, m, e
        t = t.transpose(2, 0, 3, 5, 1, 4, 6).reshape(2, npad, npad)
        got = (t[0] + 2.0 ** -c * t[1]) * 2.0 ** -sw
        assert np.all(got[n:] == 0.0) and np.all(got[:, n:] == 0.0)
        # hi keeps `bits` bits and lo as many of the rest; FP16's subnormal grid 2^-24, BF16's 2^-133
        floor = 2.0 ** (-24 - c - sw) if c else 2.0 ** -133
        err = np.abs(got[:n, :n] - ref)
        assert np.all(err <= 2.0 ** (-2 * bits) * np.abs(ref) + floor + fp64), err.max()
