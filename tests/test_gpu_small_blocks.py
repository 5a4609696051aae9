"""The 2-bit phase kernel with as few class rows a block as can be asked for: a
row of a small lattice is one or two threads, but a block has three tracker
sums to add.  Against the oracle, bit for bit, tracker included."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,rows", [(64, 1), (64, 2), (128, 1), (192, 1)])
def test_fewest_rows_a_block(L, rows, monkeypatch):
    monkeypatch.setenv("LATTICE_PATH", "phase")
    monkeypatch.setenv("LATTICE_2BIT_ROWS", str(rows))
    print(f"case small blocks L={L} rows={rows}", flush=True)
    args = (L, 0.1, 0.25, 0.5, 1.0, 0.9, 30 + L)
    g, o = lat.Lattice(*args, encoding=1), oracle.OracleLattice(*args)
    for n in (1, 5):
        g.sweep(n)
        o.sweeps(n)
        rec = g.observables()
        assert np.array_equal(g.read_state(), o.codes), n
        assert rec.ints() == o.observables().tolist(), n
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), n
