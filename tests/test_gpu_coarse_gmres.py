"""Coarsest-level GMRES steps against the oracle where the reductions change
their chunks (one chunk, a remainder, more than 64) and where the first kernel
of a step changes its form (folded blocks, matrix cores, plain GMRES on an odd
lattice), alone and in a batch; a batch whose members stop at different steps."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

# lattice, aggregates, N: odd-even entries of a coarse vector
SHAPES = [
    ((4, 4, 4, 4), (2, 2, 2, 2), 3),       # 8 sites x 6 = 48: part of one chunk
    ((8, 4, 8, 4), (2, 2, 2, 2), 9),       # 32 x 18 = 576: a remainder
    ((16, 16, 16, 8), (2, 2, 2, 2), 32),   # 1024 x 64 = 65,536: 64 chunks of 1024
    ((16, 16, 16, 12), (2, 2, 2, 2), 24),  # 1536 x 48 = 73,728: 72 chunks
    ((8, 12, 12, 12), (4, 4, 4, 4), 6),    # 2x3^3: plain GMRES, 54 x 12
]


# 12 fixed steps; FP32: 6e-8 per rounding over sums of nine 2N-blocks and twelve
# steps, times the conditioning of a twelve-column least-squares problem
@pytest.mark.parametrize("precision,bar", [(64, 1e-10), (32, 1e-4)])
@pytest.mark.parametrize("dims,agg,n", SHAPES)
def test_fixed_steps(dims, agg, n, precision, bar):
    say("case: coarse GMRES, 12 steps", dims, agg, "N", n, "precision", precision)
    import paper_1303_1377_amd as G

    p = Pair(dims, eps=0.3, seed=2, m0=-0.1, csw=1.0)
    kw = dict(levels=2, n_tv=[n], agg=[agg], sap=[(2, 2, 2, 2)], mr_steps=[2], coarse_fixed=12)
    p.o.configure(**kw)
    p.g.configure(G.default_params(precision=precision, max_rhs=3, **kw))
    v = p.vectors(0, n, 3)
    p.o.set_vectors(0, v)
    p.o.build(0)
    p.g.set_test_vectors(0, v)
    p.g.build_level(0)
    p.g.mark_setup()
    p.o.mark_setup()
    vol1, nd1 = p.o.level_size(1)
    b = F.random_vectors(vol1, nd1, 3, 4)
    want = [np.asarray(p.o.coarse_solve(1, b[q])[0]).reshape(vol1, nd1) for q in range(3)]
    e1, its = p.g.apply("COARSE_SOLVE", 1, b[0])
    assert its == 12
    say("  alone %.2e" % rel(to_np(e1).reshape(vol1, nd1), want[0]))
    assert rel(to_np(e1).reshape(vol1, nd1), want[0]) < bar
    e3, its = p.g.apply_batch("COARSE_SOLVE", 1, b)
    for q in range(3):
        err = rel(to_np(e3)[q].reshape(vol1, nd1), want[q])
        say("  batch", q, "%.2e" % err)
        assert its[q] == 12 and err < bar


@pytest.mark.parametrize("precision", [64, 32])
def test_members_stop_at_their_own_step(precision):
    """A zero and an easy right-hand side beside a hard one: each one's count and
    residual are those of a solve alone."""
    import paper_1303_1377_amd as G

    say("case: coarse GMRES, members that stop at different steps, precision", precision)
    dims = (8, 8, 8, 8)
    p = Pair(dims, eps=0.3, seed=2, m0=-0.1, csw=1.0)
    kw = dict(levels=2, n_tv=[8], agg=[(2, 2, 2, 2)], sap=[(2, 2, 2, 2)], mr_steps=[2], coarse_tol=1e-3)
    p.g.configure(G.default_params(precision=precision, max_rhs=3, **kw))
    p.g.set_test_vectors(0, p.vectors(0, 8, 3))
    p.g.build_level(0)
    p.g.mark_setup()
    vol1, nd1 = p.g.level_size(1)
    hard = F.random_vectors(vol1, nd1, 1, 4)[0]
    easy = to_np(p.g.apply("D", 1, to_np(p.g.apply("D", 1, hard)[0]))[0]).reshape(vol1, nd1)
    b = np.stack([hard, np.zeros_like(hard), easy])
    e, its = p.g.apply_batch("COARSE_SOLVE", 1, b)
    e = to_np(e).reshape(3, vol1, nd1)
    say("  counts", its)
    assert its[1] == 0 and np.abs(e[1]).max() == 0.0
    for q in (0, 2):
        one, n1 = p.g.apply("COARSE_SOLVE", 1, b[q])
        assert n1 == its[q]
        r = b[q] - to_np(p.g.apply("D", 1, e[q])[0]).reshape(vol1, nd1)
        # the even sites are solved exactly, the odd ones to the tolerance on the reduced system
        assert np.linalg.norm(r) <= 1.5e-3 * np.linalg.norm(b[q]) * 3
        assert rel(e[q], to_np(one).reshape(vol1, nd1)) < (1e-9 if precision == 64 else 1e-3)
