"""Maps on the sides around which their construction changes from a walk over
the draws to windows of 64 of them (12 and 16 for any partner, 28 and 32 for
nearest neighbours), and lattices of both in one call, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("partner", [lat.MAP_ANY, lat.MAP_NEIGHBOUR], ids=["any", "neighbour"])
@pytest.mark.parametrize("sides,n", [((8,), 3), ((12,), 21), ((16,), 2), ((28,), 17), ((32,), 1),
                                     ((4, 12, 16, 28, 32, 64), 19)])
def test_sides_around_the_walk(sides, n, partner):
    print(f"case map walk L={sides} maps={n} partner={partner}", flush=True)
    args = [(L, 0.0, 0.25, 0.5, 1.0, 1.1, 500 + L) for L in sides]
    gs = [lat.Lattice(*a) for a in args]
    lat.map_steps_batch(gs, (1 << 32) - 2, n, partner)
    for g, a in zip(gs, args):
        o = oracle.OracleLattice(*a)
        oracle.map_steps(g.L, *a[2:7], o.codes, n, start_map=(1 << 32) - 2, track=o.track,
                         nn=partner == lat.MAP_NEIGHBOUR)
        rec = g.observables()
        assert np.array_equal(g.read_state(), o.codes), g.L
        assert rec.ints() == o.observables().tolist(), g.L
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L
