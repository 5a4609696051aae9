"""Persistent launches in which threads take several calls or tasks a phase (more
than the tracker's slots hold blocks for), and unequal lattices in one launch,
each with the blocks it asks for, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


def _pair(L, enc, seed):
    args = (L, 0.1, 0.25, 0.5, 1.0, 0.9, seed)
    return lat.Lattice(*args, encoding=enc), oracle.OracleLattice(*args)


def _check(pairs):
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(pairs))([g for g, _ in pairs])):
        assert np.array_equal(g.read_state(), o.codes), g.L
        assert rec.ints() == o.observables().tolist(), g.L
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L


@pytest.mark.parametrize("L", [1028, 1452])  # 1024 blocks of 64 threads hold 1024^2 sites
def test_several_calls_a_thread(L, monkeypatch):
    print(f"case series passes L={L}", flush=True)
    monkeypatch.setenv("LATTICE_WORDS_PERSISTENT", "1")
    monkeypatch.setenv("LATTICE_WORDS_SERIES_BLOCK", "64")
    pairs = [_pair(L, 0, L)]
    for n in (2, 3):
        pairs[0][0].sweep(n)
        pairs[0][1].sweeps(n)
        _check(pairs)


@pytest.mark.parametrize("sides,enc", [((1000,) + (388,) * 7, 0), ((384,) + (100,) * 63, 0), ((2048,) + (320,) * 7, 1)],
                         ids=["bytes", "spread", "words"])
def test_unequal_lattices(sides, enc):
    print(f"case series passes {sides[0]} and {len(sides) - 1} of {sides[1]}", flush=True)
    pairs = [_pair(L, enc, 10 + i) for i, L in enumerate(sides)]
    for n in (2, 3):
        lat.sweep_batch([g for g, _ in pairs], n)
        for _, o in pairs:
            o.sweeps(n)
        _check(pairs)
