"""The tile order built on the device (recursive bisection: median selection per
segment, then counting in LDS) against the same bisection by plain sorts: the
permutation is integer and has to agree exactly.  Sizes sit on both sides of a
leaf (16 slots), of the LDS stage (512 slots), of one and two selection levels;
node sets include equal coordinates (keys decided by the node index alone) and
clumps that share a histogram digit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")

LEAF, QMAX = 16, float((1 << 24) - 1)


def _order(x):
    """Bisection by sorting every segment of every level."""
    n = len(x)
    nb = -(-n // LEAF)
    levels = 0
    while (1 << levels) < nb:
        levels += 1
    perm = np.arange(n)
    c = x.astype(np.float32).astype(np.float64)
    for l in range(levels):
        for s in range(1 << l):
            a, b = min(n, ((s * nb) >> l) * LEAF), min(n, (((s + 1) * nb) >> l) * LEAF)
            seg = perm[a:b]
            lo, ext = c[seg].min(0), c[seg].max(0) - c[seg].min(0)
            ax = int(np.argmax(ext))
            q = np.zeros(len(seg))
            if ext[ax] > 0:
                q = np.floor(np.clip((c[seg, ax] - lo[ax]) / ext[ax] * QMAX, 0.0, QMAX))
            perm[a:b] = seg[np.lexsort((seg, q))]
    return perm


def _perm_of(prob):
    up = lambda v: -(-v // 256) * 256  # noqa: E731
    off = up(16 * prob.npad) + up(8 * prob.npad) + up(24 * prob.npad) + 256
    return prob.pack[off:off + 4 * prob.npad].cpu().numpy().view(np.int32)


@pytest.mark.parametrize("n", [1, 16, 17, 40, 511, 512, 513, 1024, 1041, 2100, 9000])
@pytest.mark.parametrize("kind", ["sphere", "same", "line", "clump"])
def test_tile_order(n, kind):
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 3))
    if kind == "sphere":
        x /= np.linalg.norm(x, axis=1, keepdims=True)
    elif kind == "same":
        x[:] = 0.25                         # every key decided by the node index
    elif kind == "line":
        x = np.round(x, 1)                  # many equal coordinates
        x[:, 1:] = 0.5
    else:
        x[: 9 * n // 10] *= 1e-7            # most nodes in one digit of the first axis
    prob = P.Problem(P.Context(0), torch.from_numpy(x).cuda(), torch.ones(n, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    perm = _perm_of(prob)
    np.testing.assert_array_equal(perm[:n], _order(x))
    np.testing.assert_array_equal(perm[n:], np.arange(n, prob.npad))
