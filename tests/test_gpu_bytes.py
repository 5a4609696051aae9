"""The multi-block kernel on int8 lattices whose side is not a multiple of 64:
the smallest sides, rows of odd numbers of groups, the sides around which the
on-chip kernels end, several passes of the grid, unequal lattices in one launch,
states at any byte address and graphs, against the oracle bit for bit.
"""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat
import workloads

pytestmark = pytest.mark.gpu

SMALL = workloads.SMALL


def _pair(L, seed, T=0.9, n=0.1):
    spec = SMALL.with_(L=L, seed=seed, T=T, n=n)
    args = (spec.L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
    return lat.Lattice(*args), oracle.OracleLattice(*args)


def _check(pairs):
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(pairs))([g for g, _ in pairs])):
        assert np.array_equal(g.read_state(), o.codes), g.L
        assert rec.ints() == o.observables().tolist(), g.L
        assert [rec.track_nD, rec.track_nV, rec.track_nJ] == o.track.tolist(), g.L


@pytest.mark.parametrize("L", [4, 8, 12, 20, 36, 68, 100, 388, 444, 500, 516, 1000])
def test_sides_match_oracle(L, monkeypatch):
    monkeypatch.setenv("LATTICE_PATH", "phase")
    print(f"case bytes L={L}", flush=True)
    pairs = [_pair(L, 40 + L)]
    for n in (1, 6 if L < 600 else 2):
        pairs[0][0].sweep(n)
        pairs[0][1].sweeps(n)
        _check(pairs)


@pytest.mark.parametrize("block", [64, 256, 1024])
def test_several_passes_of_the_grid(block, monkeypatch):
    """64 threads and 2048 blocks hold 2097152 sites."""
    monkeypatch.setenv("LATTICE_WORDS_BLOCK", str(block))
    print(f"case bytes L=1452 block={block}", flush=True)
    pairs = [_pair(1452, 3)]
    pairs[0][0].sweep(1)
    pairs[0][1].sweeps(1)
    _check(pairs)


def test_unequal_lattices_in_one_call():
    print("case bytes batch", flush=True)
    pairs = [_pair(L, 60 + L) for L in (388, 508, 100, 444, 516, 64)]
    lat.sweep_batch([g for g, _ in pairs], 3)
    for _, o in pairs:
        o.sweeps(3)
    _check(pairs)
    recs = pairs[1][0].sweep_series(3, 2)
    for r in recs:
        pairs[1][1].sweeps(2)
        assert r.ints() == pairs[1][1].observables().tolist()
    _check(pairs)


def test_graph():
    print("case bytes graph", flush=True)
    pairs = [_pair(L, 80 + L) for L in (388, 500, 36)]
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


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_states_at_any_byte_address(offset):
    import torch

    L = 396
    print(f"case bytes state at byte offset {offset}", flush=True)
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


@pytest.mark.parametrize("L,enc,count", [(256, 1, 1), (256, 0, 1), (260, 0, 3), (340, 0, 1), (388, 0, 9), (388, 0, 1), (1000, 0, 1)])
def test_persistent_and_spread_calls(L, enc, count):
    """Calls on both sides of the rules that spread lattices over the chip: one
    sweep, a few, and many, in turn with reads and series."""
    print(f"case spread L={L} enc={enc} count={count}", flush=True)
    pairs = []
    for i in range(count):
        spec = SMALL.with_(L=L, seed=20 + i, T=0.6 + 0.2 * i, encoding=enc)
        args = (spec.L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
        pairs.append((lat.Lattice(*args, encoding=enc), oracle.OracleLattice(*args)))
    for n in (1, 2, 11) if L < 500 else (1, 2):
        lat.sweep_batch([g for g, _ in pairs], n)
        for _, o in pairs:
            o.sweeps(n)
        _check(pairs)
    g, o = pairs[0]
    if L < 500:
        for intervals, every in ((2, 12), (3, 1)):
            for r in g.sweep_series(intervals, every):
                o.sweeps(every)
                assert r.ints() == o.observables().tolist()
                assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist()
        g.sweep(7)
        o.sweeps(7)
        _check(pairs)


def test_on_a_stream_of_its_own():
    """No lattice spreads and none of these is persistent there; same results."""
    import torch

    print("case bytes and on-chip lattices on a stream of their own", flush=True)
    s = torch.cuda.Stream()
    for L, n in ((340, 12), (388, 6), (516, 3)):
        g = lat.Lattice(L, 0.1, 0.1, 0.5, 1.0, 1.0, 60 + L, stream=s)
        o = oracle.OracleLattice(L, 0.1, 0.1, 0.5, 1.0, 1.0, 60 + L)
        g.sweep(n)
        o.sweeps(n)
        assert np.array_equal(g.read_state(), o.codes), L
        assert g.observables().ints() == o.observables().tolist(), L
        g.destroy()
