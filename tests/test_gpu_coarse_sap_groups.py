"""Coarse SAP with right-hand sides in groups of two and four: more workgroups than
CUs (128 and 64 blocks per colour), with remainders of a group, against the
oracle."""
import pytest

from tests import test_gpu_coarse_sap as sap

pytestmark = pytest.mark.gpu

SHAPES = [
    ((16, 16, 16, 16), (2, 2, 2, 2), 6, 3),    # 128 blocks: pairs
    ((16, 16, 16, 16), (2, 2, 2, 2), 7, 8),    # fours in FP32, pairs in FP64 and FP16 (columns on 8 bytes: single)
    ((16, 16, 16, 16), (2, 2, 2, 2), 10, 7),   # fours in FP32 and FP16
    ((16, 16, 16, 16), (4, 4, 2, 2), 16, 9),   # 32 blocks of 1024 rows: pairs, FP64 with one partial row and one hop
]


@pytest.mark.parametrize("precision", [64, 32, 16])
@pytest.mark.parametrize("dims,block,n,k", SHAPES)
def test_groups(dims, block, n, k, precision):
    sap.test_coarse_sap_shapes(dims, block, n, k, precision)
