"""Persistent launches whose blocks do not come together: with
LATTICE_ASSEMBLE_TICKS=0 the first meeting calls every launch off, and the launch
behind it, a block a lattice, does the sweeps and writes the records.  Every
kind of lattice that takes a persistent launch, every number of lanes, one
counter and two levels, against the oracle, bit for bit; launches that come
together in between."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


def _pair(L, enc, seed):
    args = (L, 0.1, 0.25, 0.5, 1.0, 0.9, seed)
    return lat.Lattice(*args, encoding=enc), oracle.OracleLattice(*args)


def _same(g, o, rec):
    assert np.array_equal(g.read_state(), o.codes), g.L
    assert rec.ints() == o.observables().tolist(), g.L
    assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L


@pytest.mark.parametrize("L,enc,lanes", [(320, 1, 8), (512, 0, 8), (512, 1, 4), (576, 1, 8), (512, 1, 2), (512, 1, 1),
                                         (1088, 1, 4), (256, 1, 0), (340, 0, 0), (388, 0, 0), (1000, 0, 0)])
def test_launches_called_off(L, enc, lanes, monkeypatch):
    print(f"case assemble L={L} enc={enc} lanes={lanes}", flush=True)
    if lanes:
        monkeypatch.setenv("LATTICE_WORDS_LANES", str(lanes))
    g, o = _pair(L, enc, 20 + L)
    n = 12 if L < 400 else 2
    for ticks in ("0", None, "0"):
        if ticks is None:
            monkeypatch.delenv("LATTICE_ASSEMBLE_TICKS")
        else:
            monkeypatch.setenv("LATTICE_ASSEMBLE_TICKS", ticks)
        g.sweep(n)
        o.sweeps(n)
        _same(g, o, g.observables())
        for r in g.sweep_series(3, n):
            o.sweeps(n)
            assert r.ints() == o.observables().tolist()
            assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist()
        _same(g, o, g.observables())


@pytest.mark.parametrize("sides,enc", [((320, 512, 1024), 1), ((388, 508, 516), 0)])
def test_batches_called_off(sides, enc, monkeypatch):
    print(f"case assemble batch {sides}", flush=True)
    monkeypatch.setenv("LATTICE_ASSEMBLE_TICKS", "0")
    pairs = [_pair(L, enc, 40 + i) for i, L in enumerate(sides)]
    lat.sweep_batch([g for g, _ in pairs], 2)
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(pairs))([g for g, _ in pairs])):
        o.sweeps(2)
        _same(g, o, rec)
