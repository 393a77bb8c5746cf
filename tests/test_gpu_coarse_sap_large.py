"""Coarse SAP blocks at the limit that configure accepts (2048 rows of one parity
in table-built blocks): many sites with few unknowns, whose hop lists take most of
the LDS that FP64 fields leave."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

# lattice, level-1 aggregates and SAP blocks, test vectors: even sites x 2 N rows
SHAPES = [
    ((20, 20, 12, 12), (2, 2, 2, 1), (10, 10, 6, 3), 1),   # 900 x 2
    ((28, 12, 12, 8), (2, 2, 2, 2), (14, 6, 6, 2), 2),     # 504 x 4
]


# bars as for the smaller blocks: FP64 rounding; 1e-7 per operation over a sweep
@pytest.mark.parametrize("precision,bar", [(64, 1e-12), (32, 1e-5)])
@pytest.mark.parametrize("dims,agg,block,n", SHAPES)
def test_large_blocks(dims, agg, block, n, precision, bar):
    say("case: large coarse SAP blocks", dims, block, "N", n, "precision", precision)
    import paper_1303_1377_amd as G

    p = Pair(dims, eps=0.3, seed=5, m0=-0.1, csw=1.0)
    kw = dict(levels=3, n_tv=[n, 1], agg=[(2, 2, 2, 2), agg], sap=[(2, 2, 2, 2), block], mr_steps=[2, 3])
    p.o.configure(**kw)
    p.g.configure(G.default_params(precision=precision, max_rhs=2, **kw))
    v = p.vectors(0, n, 7)
    p.o.set_vectors(0, v)
    p.o.build(0)
    p.g.set_test_vectors(0, v)
    p.g.build_level(0)
    p.g.mark_setup()
    vol1, nd1 = p.o.level_size(1)
    b = F.random_vectors(vol1, nd1, 2, 9)
    z = to_np(p.g.apply_batch("SAP", 1, b, arg=2)[0]).reshape(2, vol1, nd1)
    for q in range(2):
        err = rel(z[q], np.asarray(p.o.sap(1, b[q], 2)).reshape(vol1, nd1))
        say("  rhs", q, "error %.2e" % err)
        assert err < bar
