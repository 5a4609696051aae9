"""Every call that returns data of a lattice whose device-wide barrier timed out
says so with LAT_EHIP: the codes, the records of a graph's replay, the penalty
sweeps, besides the observables.  Forced from the host with a bound of no time
at all (LATTICE_BARRIER_TICKS=0): every wait is up at once, and every kernel
ends.  Lattices of each kind that the persistent kernels take: the multi-block
sides, ragged int8 sides, and on-chip sides spread over the chip."""
import pytest

import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


def _fails(f, *a):
    with pytest.raises(lat.LatticeError) as e:
        f(*a)
    assert e.value.code == lat.LAT_EHIP


@pytest.mark.parametrize("L,enc", [(512, 1), (512, 0), (388, 0), (340, 0), (256, 1)])
def test_every_read_reports_a_time_out(L, enc, monkeypatch):
    print(f"case barrier reads L={L} enc={enc}", flush=True)
    monkeypatch.setenv("LATTICE_BARRIER_TICKS", "0")
    g = lat.Lattice(L, 0.1, 0.25, 0.5, 1.0, 0.9, 5, encoding=enc)
    g.sweep(20)
    monkeypatch.delenv("LATTICE_BARRIER_TICKS")
    _fails(g.read_state)
    _fails(g.observables)
    _fails(lat.BatchObservables(1), [g])
    _fails(lat.observables_batch_noalloc, [g])
    graph = lat.BatchGraph([g], 1)
    graph.launch()
    _fails(graph.read)
    graph.destroy()
    if enc == 0:
        _fails(g.mu_sweeps, 0, 2, 0.5, 0.0)
    buf = g.sweep_series(2, 1, read=False)
    _fails(g.read_series, buf, 2)
    _fails(g.read_state)
    g.destroy()


def test_one_time_out_among_many_lattices(monkeypatch):
    """The flags of several lattices are gathered, 256 a launch."""
    print("case barrier reads, 300 lattices", flush=True)
    gs = [lat.Lattice(320, 0.1, 0.25, 0.5, 1.0, 0.9, i, encoding=1) for i in range(300)]
    obs = lat.BatchObservables(300)
    lat.sweep_batch(gs, 2)
    assert len(obs(gs)) == 300
    monkeypatch.setenv("LATTICE_BARRIER_TICKS", "0")
    gs[299].sweep(20)
    monkeypatch.delenv("LATTICE_BARRIER_TICKS")
    _fails(obs, gs)
    assert len(obs(gs[:299])) == 299
    _fails(obs, gs[297:])
    _fails(obs, gs[298:])
