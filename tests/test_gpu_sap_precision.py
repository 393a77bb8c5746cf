"""Rounding of the FP32 fine SAP: the error of a sweep against the FP64 sweep must
not exceed that of the textbook order (all eight hops of a site summed before b
joins them), measured with these inputs as 1.339e-7 (4^4 blocks) and 1.307e-7
(2^4).  A norm over two vectors of this many entries is known to 0.1 %; the bars
leave 0.4 %."""
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block,bar", [((16, 16, 16, 16), 4, 1.345e-7), ((24, 12, 12, 12), 2, 1.312e-7)])
def test_fp32_sweep_error(dims, block, bar):
    import torch

    import paper_1303_1377_amd as G

    say("case: rounding of the FP32 SAP", dims, "blocks", block)
    s = G.Solver(dims, F.make_gauge_device(dims, 0.4, 1, ape_steps=2), -0.05, 1.0)
    torch.manual_seed(1)
    v = torch.randn(2, dims[0] * dims[1] * dims[2] * dims[3], 12, dtype=torch.complex128, device="cuda")
    z = {}
    for precision in (64, 32):
        s.configure(G.default_params(levels=2, n_tv=[4], agg=[(2, 2, 2, 2)], sap=[(block,) * 4], mr_steps=[4],
                                     precision=precision, max_rhs=2, outer_restart=2))
        z[precision] = s.apply_batch("SAP", 0, v, arg=2)[0].clone()
    err = float((z[32] - z[64]).norm() / z[64].norm())
    say("  error %.4e" % err)
    assert err < bar
