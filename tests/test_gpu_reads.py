"""Record reads on both sides of the sizes of the pinned blocks they come
through (24 KiB and 2 MiB, then in pieces of 1 MiB, with the error flags): series, batches and graphs of
small lattices against the oracle, and the flags of lattices that ran the
multi-block persistent kernel.
"""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat
import workloads

pytestmark = pytest.mark.gpu

SMALL = workloads.SMALL


def _pair(spec):
    args = (spec.L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
    return lat.Lattice(*args, encoding=spec.encoding), oracle.OracleLattice(*args)


def _same(rec, o, sweep):
    assert rec.ints() == o.observables().tolist()
    assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist()
    assert rec.sweep == sweep


@pytest.mark.parametrize("intervals", [1, 278, 279, 280, 400])
def test_series(intervals):
    print(f"case series read, {intervals} records", flush=True)
    g, o = _pair(SMALL.with_(L=8, seed=31))
    recs = g.sweep_series(intervals, 1)
    assert len(recs) == intervals
    for k, r in enumerate(recs):
        o.sweeps(1)
        _same(r, o, k + 1)


@pytest.mark.parametrize("count,intervals", [(1, 1), (2, 153), (2, 154), (307, 1), (308, 1), (5, 100), (230, 115)])
def test_batch_and_graph(count, intervals):
    print(f"case batch and graph reads, {count} x {intervals} records", flush=True)
    pairs = [_pair(SMALL.with_(L=8, seed=100 + i, T=0.5 + 0.01 * i)) for i in range(count)]
    gs = [g for g, _ in pairs]
    graph = lat.BatchGraph(gs, 1, intervals)
    for rep in range(2):
        graph.launch()
        rows = graph.read()
        for k in range(intervals):
            for (g, o), r in zip(pairs, rows[k]):
                o.sweeps(1)
                _same(r, o, rep * intervals + k + 1)
    for (g, o), r in zip(pairs, lat.BatchObservables(count)(gs)):
        _same(r, o, 2 * intervals)
    graph.destroy()


@pytest.mark.parametrize("small", [3, 310])
def test_flags_of_persistent_lattices(small):
    """Lattices with a device-wide barrier and without in one call."""
    print(f"case flags, {small} small lattices and 2 multi-block ones", flush=True)
    pairs = [_pair(SMALL.with_(L=8, seed=500 + i)) for i in range(small)]
    pairs.insert(1, _pair(SMALL.with_(L=320, seed=7, encoding=1)))
    pairs.append(_pair(SMALL.with_(L=320, seed=8, encoding=0)))
    gs = [g for g, _ in pairs]
    lat.sweep_batch(gs, 2)
    for (g, o), r in zip(pairs, lat.BatchObservables(len(gs))(gs)):
        o.sweeps(2)
        _same(r, o, 2)
        if g.L > 8:
            assert np.array_equal(g.read_state(), o.codes)
