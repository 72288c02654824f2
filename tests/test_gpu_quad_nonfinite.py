"""The grid of the nearest-node search over nodes whose extents are not ordinary
numbers: a coordinate that is infinite or NaN, and surfaces so small or so large that
their volume leaves FP64's range.  The cell size is found for all of them, and the
stencils of the triangles with finite vertices are the k nearest nodes."""
import numpy as np
import pytest
import torch

from oracle import quadrature as Q
from workloads import meshes
from workloads import surfaces as S

pytestmark = pytest.mark.gpu
P = pytest.importorskip("paper_2504_13379_amd")
INF, NAN = float("inf"), float("nan")


@pytest.mark.parametrize("n", [300, 1500])
@pytest.mark.parametrize("scale,odd", [(1.0, (INF, 0.0, 0.0)), (1.0, (-INF, INF, 0.3)), (1.0, (0.1, NAN, 0.2)),
                                       (1.0, (NAN, NAN, INF)), (1e-110, None), (1e120, None)])
def test_grid_of_extreme_extents(n, scale, odd):
    x = S.fibonacci_sphere(n)
    tris = meshes.triangulate(S.Surface("sphere", x, x, {}, True))
    nrm, x = x.copy(), x * scale
    if odd is not None:
        x[7] = odd
    _, st, _ = P.quad_weights(P.Context(0), torch.from_numpy(x), torch.from_numpy(nrm), tris, P.PROJ_ORIGIN, 20, details=True)
    torch.cuda.synchronize()
    keep = ~np.any(tris == 7, axis=1) if odd is not None else np.ones(len(tris), bool)
    t = tris[keep]
    far = np.where(np.isfinite(x), x, 1e150)         # never among the nearest
    cen = (x[t[:, 0]] + x[t[:, 1]] + x[t[:, 2]]) / 3.0
    np.testing.assert_array_equal(st.cpu().numpy()[keep], Q.stencils(far, cen, 20))
