"""Fine SAP against the oracle over block shapes whose hops out of the block fall
differently on the lanes: fewer than lanes, exactly one each, two each (an
extent of two beside longer ones), directions that one block spans, and blocks
whose colours meet themselves across the lattice; every storage, single and in
a batch."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

SHAPES = [
    ((4, 4, 4, 4), (2, 2, 2, 2), 4),
    ((8, 8, 8, 8), (4, 4, 4, 4), 3),
    ((8, 4, 4, 4), (2, 4, 4, 4), 3),      # two hops per lane in direction 0, none in the others
    ((4, 8, 8, 8), (4, 4, 2, 4), 2),
    ((4, 4, 8, 8), (2, 2, 4, 4), 4),
    ((4, 4, 4, 16), (2, 2, 2, 8), 3),
    ((8, 8, 4, 4), (8, 4, 2, 2), 2),
    ((12, 4, 8, 4), (2, 4, 4, 2), 0),     # no MR step
    ((4, 4, 4, 4), (4, 4, 4, 4), 3),      # no hop leaves the block
]


# FP64: rounding; FP32: 1e-7 per operation over the sums of a sweep; FP16 storage:
# 2^-11 per stored operator and vector entry
@pytest.mark.parametrize("precision,bar", [(64, 1e-12), (32, 1e-5), (16, 1e-2)])
@pytest.mark.parametrize("dims,block,mr", SHAPES)
def test_sap_block_shapes(dims, block, mr, precision, bar):
    say("case: fine SAP", dims, block, "MR", mr, "precision", precision)
    import paper_1303_1377_amd as G

    p = Pair(dims, eps=0.3, seed=4, m0=-0.1, csw=1.0)
    kw = dict(levels=2, n_tv=[2], agg=[(2, 2, 2, 2)], sap=[block], mr_steps=[mr])
    p.o.configure(**kw)
    p.g.configure(G.default_params(precision=precision, max_rhs=2, **kw))
    b = F.gaussian_spinor(dims, 6, nrhs=2)
    z = to_np(p.g.apply_batch("SAP", 0, b.reshape(2, p.vol, 12), arg=2)[0]).reshape(b.shape)
    for q in range(2):
        err = rel(z[q], np.asarray(p.o.sap(0, b[q], 2)).reshape(b[q].shape))
        say("  rhs", q, "error %.2e" % err)
        assert err < bar
