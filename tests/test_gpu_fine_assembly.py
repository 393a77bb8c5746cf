"""D_c = P^H D P of the finest level against the oracle, over aggregates whose
faces fill part of a wave, exactly one and several, on both sides of the 256
sites that separate the two compiled forms, with one aggregate across the
lattice and with an extent of one."""
import pytest

from tests._gpu import Pair, rel, say, to_np

pytestmark = pytest.mark.gpu

SHAPES = [((4, 4, 4, 4), (1, 2, 2, 2), 1), ((12, 4, 4, 4), (3, 2, 2, 2), 5), ((8, 8, 4, 4), (4, 4, 2, 1), 7),
          ((12, 12, 4, 4), (6, 6, 2, 2), 4), ((8, 8, 8, 8), (4, 4, 4, 4), 32), ((8, 8, 8, 8), (8, 4, 4, 4), 6),
          ((16, 8, 8, 8), (8, 4, 4, 4), 3), ((8, 8, 8, 16), (4, 4, 8, 8), 2)]


# FP64: rounding; FP32: 6e-8 per operation through the orthonormalisation and the hops
@pytest.mark.parametrize("precision,bar", [(64, 1e-12), (32, 1e-5)])
@pytest.mark.parametrize("dims,agg,n", SHAPES)
def test_fine_assembly(dims, agg, n, precision, bar):
    say("case: fine assembly", dims, "aggregate", agg, "N", n, "precision", precision)
    p = Pair(dims, eps=0.35, seed=4, m0=-0.25, csw=1.0)
    p.configure(precision=precision, levels=2, n_tv=[n], agg=[agg], sap=[(2, 2, 2, 2)], mr_steps=[2])
    tv = p.vectors(0, n, 2)
    p.o.set_vectors(0, tv)
    p.o.build(0)
    p.g.set_test_vectors(0, tv)
    p.g.build_level(0)
    M, Mo = to_np(p.g.get_coarse(1)[0]), p.o.get_coarse(1)[0]
    for slot in range(9):
        e = rel(M[:, slot], Mo[:, slot]) if abs(Mo[:, slot]).max() else abs(M[:, slot]).max()
        assert e < bar, (slot, e)
