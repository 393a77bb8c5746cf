"""Coarse-level SAP against the oracle where its split of a block over lane
groups, rows per lane and right-hand-side groups changes: block shapes from the
layout and from tables, unknowns per site that leave remainders, and batches on
both sides of every group width."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F

from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

# lattice, level-1 SAP blocks, test vectors N (2N unknowns per site), batch
SHAPES = [
    ((8, 8, 8, 8), (2, 2, 2, 2), 1, 1),      # one lane per column in FP16 / FP32
    ((8, 8, 8, 8), (2, 2, 2, 2), 7, 3),      # 14 unknowns: FP16 columns on 8-byte boundaries
    ((8, 8, 8, 8), (2, 2, 2, 2), 20, 5),
    ((16, 16, 16, 8), (2, 2, 2, 2), 20, 4),  # 128 blocks per colour: groups of four (FP64: of two)
    ((16, 16, 16, 8), (2, 2, 2, 2), 13, 2),
    ((8, 8, 8, 8), (4, 4, 4, 4), 4, 3),      # 128 even sites, one block per colour and direction
    ((8, 12, 12, 12), (2, 3, 3, 3), 20, 2),  # tables, 27 even sites
    ((12, 24, 24, 24), (6, 6, 6, 6), 1, 1),  # 648 even sites of 2 unknowns: FP64 finds neighbours again
    ((8, 12, 12, 12), (2, 3, 3, 3), 32, 1),  # 64 unknowns: a site needs more lanes than a part has
]
# FP64: rounding; FP32: 1e-7 per operation over the sums of a sweep; FP16 storage:
# 2^-11 per operator entry, summed over the nine blocks of a site
BARS = {64: 1e-12, 32: 1e-5, 16: 1e-2}


@pytest.mark.parametrize("precision", [64, 32, 16])
@pytest.mark.parametrize("dims,block,n,k", SHAPES)
def test_coarse_sap_shapes(dims, block, n, k, precision):
    say("case: coarse SAP", dims, block, "N", n, "batch", k, "precision", precision)
    import paper_1303_1377_amd as G

    p = Pair(dims, eps=0.3, seed=5, m0=-0.1, csw=1.0)
    kw = dict(levels=3, n_tv=[n, 1], agg=[(2, 2, 2, 2), (2, 2, 2, 2)], sap=[(2, 2, 2, 2), block], mr_steps=[2, 3])
    p.o.configure(**kw)
    p.g.configure(G.default_params(precision=precision, max_rhs=k, **kw))
    v = p.vectors(0, n, 7)
    p.o.set_vectors(0, v)
    p.o.build(0)
    p.g.set_test_vectors(0, v)
    p.g.build_level(0)
    p.g.mark_setup()
    vol1, nd1 = p.o.level_size(1)
    b = F.random_vectors(vol1, nd1, k, 9)
    z, _ = p.g.apply_batch("SAP", 1, b, arg=2)
    z = to_np(z).reshape(k, vol1, nd1)
    for q in range(k):
        err = rel(z[q], np.asarray(p.o.sap(1, b[q], 2)).reshape(vol1, nd1))
        say("  rhs", q, "error %.2e" % err)
        assert err < BARS[precision]
