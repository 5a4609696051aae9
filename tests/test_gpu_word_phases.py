"""The multi-block kernel of one launch per phase on batches of unequal
lattices (rows of the grid with different numbers of blocks, lattices that are
through with their sweeps before others), every block size, and replayed from a
graph, against the oracle bit for bit.
"""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat
import workloads

pytestmark = pytest.mark.gpu

SMALL = workloads.SMALL


def _pairs():
    out = []
    for L, enc in ((64, 1), (320, 0), (448, 1), (128, 1)):
        spec = SMALL.with_(L=L, encoding=enc, seed=900 + L, T=0.7 + L / 1000)
        args = (spec.L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
        out.append((lat.Lattice(*args, encoding=enc), oracle.OracleLattice(*args)))
    return out


def _check(pairs):
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(pairs))([g for g, _ in pairs])):
        assert np.array_equal(g.read_state(), o.codes), g.L
        assert rec.ints() == o.observables().tolist(), g.L
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L


@pytest.mark.parametrize("block", [64, 192, 256, 320, 1024])
@pytest.mark.parametrize("lanes", [1, 2, 4, 8])
def test_unequal_lattices(block, lanes, monkeypatch):
    monkeypatch.setenv("LATTICE_PATH", "words")
    monkeypatch.setenv("LATTICE_WORDS_PERSISTENT", "0")
    monkeypatch.setenv("LATTICE_WORDS_BLOCK", str(block))
    monkeypatch.setenv("LATTICE_WORDS_PHASE_LANES", str(lanes))
    print(f"case word phases block={block} lanes={lanes}", flush=True)
    pairs = _pairs()
    lat.sweep_batch([g for g, _ in pairs], 3)
    for _, o in pairs:
        o.sweeps(3)
    _check(pairs)


def test_replayed_from_a_graph(monkeypatch):
    monkeypatch.setenv("LATTICE_PATH", "words")
    print("case word phases in a graph", flush=True)
    pairs = _pairs()
    graph = lat.BatchGraph([g for g, _ in pairs], 2, 2)
    for _ in range(3):
        graph.launch()
        rows = graph.read()
        for k in range(2):
            for (_, o), rec in zip(pairs, rows[k]):
                o.sweeps(2)
                assert rec.ints() == o.observables().tolist()
        for g, o in pairs:  # eager work between the replays
            g.sweep(1)
            o.sweeps(1)
        _check(pairs)
    graph.destroy()
