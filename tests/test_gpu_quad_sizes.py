"""Quadrature weights at the edges of the kernels' ranges against the FP64 oracle:
stencil sizes on both sides of each register size of the element solve (20, 32,
45, 57) and the smallest one, and nodes clumped so that a cell neighbourhood
holds from a few to well over 512 nodes, so that the one-pass nearest-node search
and the ring search both run, and nodes' entry lists of very different lengths.

Tolerance: stencils exactly; weights to 1e-10 of max|q|, as the other weight tests
(both sides solve the same FP64 systems, whose conditioning costs about 1e-12)."""
import numpy as np
import pytest
import torch

from oracle import quadrature as Q
from workloads import meshes
from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")
TOL = 1e-10


def _surface(n, shift):
    x = S.fibonacci_sphere(n)
    x[:, 2] += shift                        # nodes crowd about one pole
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    return S.Surface("sphere", x, x, {}, True)


@pytest.mark.parametrize("n,k,shift", [(300, 6, 0.0), (400, 20, 0.0), (500, 33, 0.0), (700, 45, 0.0), (700, 46, 0.0),
                                       (3000, 32, 0.6), (6000, 20, 0.95), (6000, 57, 0.8)])
def test_quad_weights_sizes(n, k, shift):
    surf = _surface(n, shift)
    tris = meshes.triangulate(surf)
    q, st, _ = P.quad_weights(P.Context(0), torch.from_numpy(surf.xyz), torch.from_numpy(surf.normals), tris,
                              P.PROJ_ORIGIN, k, details=True)
    torch.cuda.synchronize()
    x = surf.xyz
    cen = (x[tris[:, 0]] + x[tris[:, 1]] + x[tris[:, 2]]) / 3.0
    np.testing.assert_array_equal(st.cpu().numpy(), Q.stencils(x, cen, k))
    q_ref = Q.surface_weights(surf, k=k)
    err = np.max(np.abs(q.cpu().numpy() - q_ref)) / np.max(np.abs(q_ref))
    assert err <= TOL, err
