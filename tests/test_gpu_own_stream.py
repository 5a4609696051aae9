"""On a stream of the caller's own no call takes a persistent launch, also where the
environment asks for one: with a bound of no time for its barriers
(LATTICE_BARRIER_TICKS=0) a persistent launch would leave the state invalid, and
the codes, records and tracker equal the oracle's."""
import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("asked", [False, True], ids=["default", "asked"])
@pytest.mark.parametrize("L,enc", [(320, 1), (512, 0), (1024, 1), (1088, 1), (388, 0), (256, 1), (340, 0), (2112, 1)])
def test_no_persistent_launch(L, enc, asked, monkeypatch):
    import torch

    print(f"case own stream L={L} enc={enc} asked={asked}", flush=True)
    monkeypatch.setenv("LATTICE_BARRIER_TICKS", "0")
    if asked:
        monkeypatch.setenv("LATTICE_WORDS_PERSISTENT", "1")
        monkeypatch.setenv("LATTICE_PERSISTENT", "1")
    s = torch.cuda.Stream()
    args = (L, 0.1, 0.25, 0.5, 1.0, 0.9, 90 + L)
    g, o = lat.Lattice(*args, encoding=enc, stream=s), oracle.OracleLattice(*args)
    n = 8 if L < 400 else 2
    g.sweep(n)
    o.sweeps(n)
    assert np.array_equal(g.read_state(), o.codes)
    with torch.cuda.stream(s):
        lat.sweep_batch([g], n)
        recs = g.sweep_series(2, 1)
    o.sweeps(n)
    for r in recs:
        o.sweeps(1)
        assert r.ints() == o.observables().tolist()
        assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist()
    assert np.array_equal(g.read_state(), o.codes)
    assert g.observables().ints() == o.observables().tolist()
