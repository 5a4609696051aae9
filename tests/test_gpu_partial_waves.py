"""The cooperative form of the 2-bit phase path (LATTICE_PERSISTENT=1) in blocks
whose last wave has one or two lanes: rows x W threads with W = L / 64 words a
class row.  Every wave of a block has to take the same schedule: against the
oracle, bit for bit, tracker included."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,rows", [
    (64, 1),    # one lane
    (64, 2),    # two lanes, two rows
    (128, 1),   # two lanes, one row
    (4160, 1),  # 65 words a row: a whole wave and one lane
    (4224, 1),  # 66: a whole wave and two lanes
])
def test_last_wave_of_one_or_two_lanes(L, rows, monkeypatch):
    monkeypatch.setenv("LATTICE_PATH", "phase")
    monkeypatch.setenv("LATTICE_PERSISTENT", "1")
    monkeypatch.setenv("LATTICE_2BIT_ROWS", str(rows))
    print(f"case partial waves L={L} rows={rows}", flush=True)
    args = (L, 0.1, 0.25, 0.5, 1.0, 0.9, 70 + L)
    g, o = lat.Lattice(*args, encoding=1), oracle.OracleLattice(*args)
    for n in (1, 5) if L < 1000 else (1, 2):
        g.sweep(n)
        o.sweeps(n)
        rec = g.observables()
        assert np.array_equal(g.read_state(), o.codes), n
        assert rec.ints() == o.observables().tolist(), n
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), n
