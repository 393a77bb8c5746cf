"""The matrix-core coarse stencil with at most 16 unknowns per site (one row tile):
its forms of one, two and four instruction steps and the lines between its two
workgroup forms there, against the FP64 product as for more unknowns."""
import pytest

from tests import test_gpu_coarse_mfma as mfma

pytestmark = pytest.mark.gpu

MEDIUM = (12, 12, 12, 12)   # 1296 sites, 648 of one parity
SHAPES = [(mfma.SMALL, 2, 3), (MEDIUM, 1, 2), (MEDIUM, 4, 4), (MEDIUM, 6, 8), (mfma.LARGE, 1, 16), (mfma.LARGE, 2, 5),
          (mfma.LARGE, 4, 9), (mfma.LARGE, 6, 2), (mfma.LARGE, 8, 8), (mfma.LARGE, 8, 3)]


@pytest.mark.parametrize("precision,bar", [(32, 2e-6), (16, 4e-3)])
@pytest.mark.parametrize("dims,n,k", SHAPES)
def test_few_unknowns(dims, n, k, precision, bar):
    mfma.test_mfma_shapes(dims, n, k, precision, bar)
