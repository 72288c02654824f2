"""Sums that are meant to be the same bit for bit.  The sources that count lie in one
group of 64 nodes or one tile of 256, so a node's FP64 total has one term that is not 0
and shows the FP32 sum itself: of a tile pair split into its source groups against the
same pair taken whole (in a problem with more tiles behind it), row and column sums; and
of the multi-state sum with its products on the matrix cores against the vector units."""
import numpy as np
import pytest
import torch

from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0, torch.cuda.Stream())


def _kernel(kind):
    return P.kernel_struct(kind, *((1.0, 0.15, 0.5, 0.4) if kind == 0 else (2.0, 0.1, 1.0, 0.3)))


def _nodes(n, rng, period):
    x = S.fibonacci_sphere(n)[rng.permutation(n)]
    if period:
        x[:, 2] = 0.0
    return x


# tiles of the problem with split pairs, first and past-the-end node of the sources
@pytest.mark.parametrize("nt,lo,hi", [(32, 31 * 256 + 64, 31 * 256 + 128), (32, 20 * 256, 21 * 256), (25, 24 * 256, 24 * 256 + 64),
                                      (25, 7 * 256, 8 * 256), (27, 23 * 256 + 192, 24 * 256)])
@pytest.mark.parametrize("kind,period", [(0, 0.0), (1, 0.0), (0, 4.0)])
def test_split_and_whole_pairs(ctx, nt, lo, hi, kind, period):
    n, more = 256 * nt, 256 * 53                 # no pair of 53 tiles is split
    rng = np.random.default_rng(lo)
    x = _nodes(more, rng, period)
    q = np.zeros(more)
    q[lo:hi] = rng.uniform(0.2, 1.0, size=hi - lo)
    u = rng.normal(0.2, 0.4, size=(1, more))
    got = []
    for m in (n, more):
        prob = P.Problem(ctx, torch.from_numpy(x[:m].copy()).cuda(), torch.from_numpy(q[:m].copy()).cuda(), period=period)
        v = torch.from_numpy(u[:, :m].copy()).cuda()
        y = prob.apply(_kernel(kind), P.Firing(20.0, 0.2), v)
        ctx.stream.synchronize()
        got.append(y.cpu().numpy()[0, :n])
    # the tiles behind a whole tile of sources take it in one column sum, the others group by group
    own = slice(hi if hi - lo == 256 else 0, None)
    assert np.all(got[0][own] != 0.0)
    np.testing.assert_array_equal(got[0][own], got[1][own])


@pytest.mark.parametrize("kind,period", [(0, 0.0), (1, 0.0), (0, 4.0)])
def test_matrix_core_and_vector_products(ctx, kind, period):
    n = 1500
    rng = np.random.default_rng(kind)
    x = _nodes(n, rng, period)
    q = np.zeros(n)
    q[512:768] = rng.uniform(-0.2, 1.0, size=256)
    u = torch.from_numpy(rng.normal(0.2, 0.4, size=(64, n))).cuda()
    prob = P.Problem(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), period=period)
    parts = [prob.apply(_kernel(kind), P.Firing(20.0, 0.2), u[b:b + 8]) for b in range(0, 64, 8)]
    ctx.stream.synchronize()
    vec = torch.cat(parts)
    for B in (9, 17, 33, 64):
        y = prob.apply(_kernel(kind), P.Firing(20.0, 0.2), u[:B])
        ctx.stream.synchronize()
        assert torch.equal(y, vec[:B]), B
