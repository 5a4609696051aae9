"""GPU parity of the persistent multi-block word kernel over its launch shapes
(lanes per a-word, block sizes, one-counter and two-level barriers, one and
several tasks a thread, lattices with barriers of their own in one launch)
against the oracle, bit for bit."""
import sys

import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat
import workloads

pytestmark = pytest.mark.gpu

SMALL = workloads.SMALL


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _pair(spec):
    args = (spec.L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
    return lat.Lattice(*args, encoding=spec.encoding), oracle.OracleLattice(*args)


def _same(g, o, rec, where):
    assert np.array_equal(g.read_state(), o.codes), where
    assert rec.ints() == o.observables().tolist(), where
    assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), where


@pytest.mark.parametrize("L,lanes,block", [
    (320, 8, 64),     # 100 blocks: two levels
    (512, 8, 256),    # 64 blocks: one counter
    (576, 8, 256),    # 81 blocks, 9 words a class row
    (576, 1, 64), (1024, 2, 256), (1024, 4, 512), (1024, 8, 512),
    (1088, 4, 512),   # just above the largest one-counter side, 17 words a row
    (2048, 4, 512), (2048, 1, 64), (2048, 8, 64),  # 1024 blocks: more than one task a thread
])
def test_shapes_match_oracle(L, lanes, block, monkeypatch):
    monkeypatch.setenv("LATTICE_WORDS_PERSISTENT", "1")
    monkeypatch.setenv("LATTICE_WORDS_LANES", str(lanes))
    monkeypatch.setenv("LATTICE_WORDS_SERIES_BLOCK", str(block))
    _say(f"case word shape L={L} lanes={lanes} block={block}")
    g, o = _pair(SMALL.with_(L=L, encoding=1, seed=60 + L, T=0.9))
    g.sweep(2)
    o.sweeps(2)
    _same(g, o, g.observables(), "plain sweeps")
    for k, r in enumerate(g.sweep_series(3, 1) + g.sweep_series(1, 2)):
        o.sweeps(1 if k < 3 else 2)
        assert r.ints() == o.observables().tolist(), k
        assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist(), k
    _same(g, o, g.observables(), "after the series")


@pytest.mark.parametrize("sides", [(320, 512, 1024), (2048, 320), (512,) * 9 + (576,) * 8],
                         ids=["mixed", "large-small", "many"])
def test_batches_match_oracle(sides):
    """Lattices of one launch meet at barriers of their own."""
    _say(f"case word batch {sides}")
    pairs = [_pair(SMALL.with_(L=L, encoding=i % 2, seed=300 + i, T=0.5 + 0.1 * i)) for i, L in enumerate(sides)]
    gs = [g for g, _ in pairs]
    for n in (1, 2):
        lat.sweep_batch(gs, n)
        for i, ((g, o), rec) in enumerate(zip(pairs, lat.BatchObservables(len(gs))(gs))):
            o.sweeps(n)
            _same(g, o, rec, f"lattice {i}")


@pytest.mark.parametrize("L", [512, 2048])
def test_captured_sweeps_replay(L):
    """A call captured into a graph takes one launch per phase; replays (with
    eager work in between) go on from the device's sweep index."""
    import torch

    _say(f"case captured sweeps L={L}")
    g, o = _pair(SMALL.with_(L=L, encoding=1, seed=90 + L, T=1.1))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        lat.sweep_batch([g], 2, stream=torch.cuda.current_stream())
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        o.sweeps(2)
        assert np.array_equal(g.read_state(), o.codes), f"replay {k}"
        lat.sweep_batch([g], 1)
        torch.cuda.synchronize()
        o.sweeps(1)
        assert np.array_equal(g.read_state(), o.codes), f"eager sweep {k}"
