"""One state on the symmetric kernel, as test_gpu_sym_rest, where the split tile pairs
lie in three, four and five rows of the order: 25, 35 and 27 tiles."""
import pytest

from .test_gpu_sym_rest import ctx, test_split_pairs as split_pairs  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kind,period", [(6400, 0, 0.0), (8900, 1, 0.0), (6700, 0, 4.0)])
def test_three_to_five_rows(ctx, n, kind, period):  # noqa: F811
    split_pairs(ctx, n, kind, period)
