"""Coarse stencil on the matrix cores against the FP64 product with the level's
own blocks (get_coarse; their assembly is compared with the oracle elsewhere):
unknowns per site on both sides of every compiled number of instruction steps, batches on both sides
of every staged width (4, 8, 16 columns), and lattices below and above the line
between its two workgroup forms; the Schur complement runs its form with the
self-block inverse."""
import numpy as np
import pytest

from paper_1303_1377_amd import fields as F
from tests._gpu import rel, say, to_np

pytestmark = pytest.mark.gpu

SMALL, LARGE = (8, 8, 8, 4), (16, 16, 16, 16)   # 128 and 4096 coarse sites (64 and 2048 of one parity)
SHAPES = [(SMALL, 1, 2), (SMALL, 8, 4), (SMALL, 10, 5), (SMALL, 13, 8), (SMALL, 16, 9), (SMALL, 19, 3), (SMALL, 20, 4),
          (SMALL, 20, 16), (SMALL, 24, 2), (SMALL, 32, 12), (LARGE, 3, 4), (LARGE, 20, 3), (LARGE, 9, 6), (LARGE, 5, 11)]


# FP32: 6e-8 per rounding over the nine 2N-blocks of a site; FP16 storage: 2^-11
# per stored entry and per rounded input over the same sum.  The Schur complement
# chains three such products.
@pytest.mark.parametrize("precision,bar", [(32, 2e-6), (16, 4e-3)])
@pytest.mark.parametrize("dims,n,k", SHAPES)
def test_mfma_shapes(dims, n, k, precision, bar):
    say("case: matrix-core coarse stencil", dims, "N", n, "batch", k, "precision", precision)
    import paper_1303_1377_amd as G

    g = G.Solver(dims, F.make_gauge(dims, 0.3, 3), -0.1, 1.0)
    g.configure(G.default_params(precision=precision, max_rhs=k, levels=2, n_tv=[n], agg=[(2, 2, 2, 2)],
                                 sap=[(2, 2, 2, 2)], mr_steps=[2]))
    vol = int(np.prod(dims))
    g.set_test_vectors(0, F.random_vectors(vol, 12, n, 3))
    g.build_level(0)
    g.mark_setup()
    vol1, nd1 = g.level_size(1)
    M, Mi = (to_np(a) for a in g.get_coarse(1))
    cd = g.level_info(1)[0]
    x = np.stack(np.unravel_index(np.arange(vol1), cd))
    odd = (x.sum(0) % 2).astype(bool)

    def hops(v):
        out = np.zeros_like(v)
        for s in range(8):
            y = x.copy()
            y[s % 4] = (y[s % 4] + (1 if s < 4 else -1)) % cd[s % 4]
            out += np.einsum("xij,xj->xi", M[:, 1 + s], v[np.ravel_multi_index(tuple(y), cd)])
        return out

    def schur(v):
        v = np.where(odd[:, None], v, 0)
        t = np.where(odd[:, None], 0, np.einsum("xij,xj->xi", Mi, hops(v)))
        return np.where(odd[:, None], np.einsum("xij,xj->xi", M[:, 0], v) - hops(t), 0)

    b = F.random_vectors(vol1, nd1, k, 4)
    y = to_np(g.apply_batch("D", 1, b)[0]).reshape(k, vol1, nd1)
    z = to_np(g.apply_batch("SCHUR", 1, b)[0]).reshape(k, vol1, nd1)
    for q in range(k):
        e = rel(y[q], np.einsum("xij,xj->xi", M[:, 0], b[q]) + hops(b[q]))
        es = rel(z[q], schur(b[q]))
        say("  rhs", q, "D %.2e Schur %.2e" % (e, es))
        assert e < bar and es < 5 * bar
