"""Canonical spinors to and from the block layout: blocks from 16 to 256 sites,
lattices whose last 256-site workgroup is partly filled, one vector and a
batch.  The round trip keeps every bit that the storage holds; D on the same
vectors agrees with the oracle, so the sites are the right ones."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

SHAPES = [((4, 4, 2, 2), (2, 2, 2, 2), (2, 2, 1, 1)), ((4, 4, 12, 2), (2, 2, 2, 2), (2, 2, 2, 1)),
          ((4, 20, 2, 4), (4, 2, 2, 4), (2, 2, 1, 2)), ((8, 4, 4, 4), (8, 2, 4, 4), (4, 2, 2, 2)),
          ((8, 8, 8, 4), (4, 4, 4, 4), (2, 2, 2, 2))]


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("dims,block,agg", SHAPES)
def test_layout_round_trip(dims, block, agg, precision):
    say("case: spinor layout", dims, "block", block, "precision", precision)
    import paper_1303_1377_amd as G

    p = Pair(dims, eps=0.3, seed=5, m0=-0.1, csw=1.0)
    p.g.configure(G.default_params(precision=precision, max_rhs=3, levels=2, n_tv=[3], agg=[agg], sap=[block], mr_steps=[2]))
    v = F.random_vectors(p.vol, 12, 3, 9)
    p.g.set_test_vectors(0, v)
    back = to_np(p.g.get_test_vectors(0)).reshape(v.shape)
    assert np.array_equal(back, v if precision == 64 else v.astype(np.complex64).astype(np.complex128))
    # rounding over the nine terms of a site (FP64; FP32)
    for op, bar in (("D", 1e-13), ("D_PREC", 1e-13 if precision == 64 else 2e-6)):
        y = to_np(p.g.apply_batch(op, 0, v)[0]).reshape(v.shape)
        for q in range(3):
            assert rel(y[q], np.asarray(p.o.apply(v[q])).reshape(v[q].shape)) < bar, (op, q)
