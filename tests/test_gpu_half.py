"""The half-byte on-chip form (sides above 384 up to 512): single lattices asked onto
the chip, in both encodings, mixed with smaller ones, at any byte address, with
records from the kernel; and as many lattices as compute units, which take it by
themselves.  Against the oracle, bit for bit."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


def _pair(L, enc, seed, T=0.9):
    args = (L, 0.1, 0.25, 0.5, 1.0, T, seed)
    return lat.Lattice(*args, encoding=enc), oracle.OracleLattice(*args)


def _check(pairs):
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(pairs))([g for g, _ in pairs])):
        assert np.array_equal(g.read_state(), o.codes), g.L
        assert rec.ints() == o.observables().tolist(), g.L
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L


@pytest.mark.parametrize("L,enc", [(388, 0), (444, 0), (448, 1), (500, 0), (508, 0), (512, 1), (512, 0)])
def test_asked_onto_the_chip(L, enc, monkeypatch):
    print(f"case half L={L} enc={enc}", flush=True)
    monkeypatch.setenv("LATTICE_PATH", "lds")
    g, o = _pair(L, enc, L)
    for n in (1, 17):
        g.sweep(n)
        o.sweeps(n)
        _check([(g, o)])
    for r in g.sweep_series(3, 2):
        o.sweeps(2)
        assert r.ints() == o.observables().tolist()
        assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist()
    _check([(g, o)])


def test_mixed_sides_and_graph(monkeypatch):
    print("case half, mixed sides", flush=True)
    monkeypatch.setenv("LATTICE_PATH", "lds")
    pairs = [_pair(L, enc, 40 + i, 0.4 + 0.2 * i) for i, (L, enc) in enumerate([(4, 0), (500, 0), (64, 1), (388, 0), (100, 0), (512, 1)])]
    lat.sweep_batch([g for g, _ in pairs], 2)
    for _, o in pairs:
        o.sweeps(2)
    _check(pairs)
    graph = lat.BatchGraph([g for g, _ in pairs], 1, 2)
    for _ in range(2):
        graph.launch()
        for row in graph.read():
            for (_, o), rec in zip(pairs, row):
                o.sweeps(1)
                assert rec.ints() == o.observables().tolist()
                assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist()
        _check(pairs)
    graph.destroy()


@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
def test_a_compute_unit_each(graph):
    """More lattices than the rule's limit: 150 of L = 388 and 396, and 130 of them
    beside one whose side the form does not take."""
    print(f"case half, 150 lattices graph={graph}", flush=True)
    pairs = [_pair(388 + 8 * (i % 2), 0, 200 + i, 0.3 + 0.01 * i) for i in range(150)]
    gs = [g for g, _ in pairs]
    if graph:
        replay = lat.BatchGraph(gs, 1, 2)
        replay.launch()
        rows = replay.read()
        for row in rows:
            for (_, o), rec in list(zip(pairs, row))[::13]:
                o.sweeps(1)
                assert rec.ints() == o.observables().tolist()
        replay.destroy()
        _check(pairs[::13])
        return
    lat.sweep_batch(gs, 2)
    for _, o in pairs[::13]:
        o.sweeps(2)
    _check(pairs[::13])
    big = _pair(516, 0, 9)
    lat.sweep_batch([big[0]] + gs[:130], 1)
    big[1].sweeps(1)
    for _, o in pairs[:130:13]:
        o.sweeps(1)
    _check([big] + pairs[:130:13])


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_states_at_any_byte_address(offset, monkeypatch):
    import torch

    L = 396
    print(f"case half, state at byte offset {offset}", flush=True)
    monkeypatch.setenv("LATTICE_PATH", "lds")
    o = oracle.OracleLattice(L, 0.1, 0.1, 0.5, 1.0, 1.0, 8)
    buf = torch.full((L * L + 64,), 0x55, dtype=torch.uint8, device="cuda")
    scratch = torch.empty(lat.scratch_bytes(L, 0), dtype=torch.uint8, device="cuda")
    p = lat.LatParams(L=L, encoding=0, n=0.1, Delta=0.1, V=0.5, J=1.0, T=1.0, seed=8, n_charged=-1, start_sweep=0,
                      init_codes=None)
    h = ctypes.c_void_p()
    lib = lat.lib()
    assert lib.lattice_create(ctypes.byref(p), buf.data_ptr() + 32 + offset, L * L, scratch.data_ptr(), scratch.numel(),
                              torch.cuda.current_stream().cuda_stream, ctypes.byref(h)) == 0
    assert lib.lattice_sweep(h, 3) == 0
    torch.cuda.synchronize()
    o.sweeps(3)
    got = buf.cpu().numpy()
    assert np.array_equal(got[32 + offset:32 + offset + L * L].astype(np.int8), o.codes)
    assert (got[:32 + offset] == 0x55).all() and (got[32 + offset + L * L:] == 0x55).all()
    assert lib.lattice_destroy(h) == 0
