"""GPU parity of the on-chip kernel that takes four pairs a thread (sides that are
a multiple of 16, the largest of a launch from 80 on) at the edges of its shapes,
against the oracle bit for bit: one task a thread and several, rows of 1 to 23
words, the smallest and the largest side, every block size, states at any byte
address, and whole observation series in one launch.  Sides of 48 and 64 stand
for the launches below the rule.
"""
import ctypes
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


@pytest.mark.parametrize("threads", [0, 64, 256, 1024])
@pytest.mark.parametrize("L", [48, 64, 80, 128, 144, 176, 192, 256, 368])
def test_sides_and_block_sizes_match_oracle(L, threads, monkeypatch):
    """17 sweeps cross the boundary between two sets of schedule words."""
    monkeypatch.setenv("LATTICE_PATH", "lds")
    if threads:
        monkeypatch.setenv("LATTICE_BATCH_THREADS", str(threads))
    _say(f"case quad form L={L} threads={threads}")
    n = 17 if L < 200 else 5
    pairs = [_pair(SMALL.with_(L=L, n=n0, T=T, seed=700 + L)) for n0, T in ((0.1, 0.8), (-0.3, 0.4))]
    pairs += [_pair(SMALL.with_(L=side, T=1.3, seed=702 + L)) for side in (16, 32, 48)]  # in the same launch
    if L % 64 == 0:
        pairs.append(_pair(SMALL.with_(L=L, T=1.7, seed=701 + L, encoding=1)))
    gs = [g for g, _ in pairs]
    lat.sweep_batch(gs, n)
    for (g, o), rec in zip(pairs, lat.BatchObservables(len(gs))(gs)):
        o.sweeps(n)
        _same(g, o, rec, f"L={L} threads={threads}")


@pytest.mark.parametrize("L,enc,intervals,every", [
    (48, 0, 40, 1), (64, 1, 35, 1), (64, 0, 9, 10), (96, 0, 7, 5), (128, 1, 5, 17), (256, 1, 4, 3), (208, 0, 3, 2),
    (48, 0, 3, 6000),  # more sweeps than one launch holds
], ids=lambda v: str(v))
def test_series_and_graph_records_match_oracle(L, enc, intervals, every):
    _say(f"case quad series L={L} enc={enc} intervals={intervals} every={every}")
    spec = SMALL.with_(L=L, encoding=enc, seed=800 + L, T=0.9)
    (g, o), (h, _) = _pair(spec), _pair(spec)
    graph = lat.BatchGraph([h], every, intervals)
    done = 0
    for rep in range(2):
        recs = g.sweep_series(intervals, every)
        graph.launch()
        for k, (r, (q,)) in enumerate(zip(recs, graph.read())):
            o.sweeps(every)
            done += every
            assert r.ints() == o.observables().tolist(), k
            assert [r.track_nD, r.track_nV, r.track_nJ] == o.track.tolist(), k
            assert r.sweep == done
            assert q.as_dict() == r.as_dict(), k
        _same(g, o, g.observables(), f"series {rep}")
        g.sweep(1)  # eager work between the replays
        h.sweep(1)
        o.sweeps(1)
        done += 1
        _same(h, o, h.observables(), f"graph {rep}")
        assert np.array_equal(g.read_state(), o.codes)
    graph.destroy()


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_states_at_any_byte_address(offset):
    """An int8 state is a byte buffer: the caller may place it anywhere."""
    import torch

    L, spec = 96, SMALL.with_(L=96, seed=77)
    _say(f"case quad state at byte offset {offset}")
    o = oracle.OracleLattice(L, spec.n, spec.Delta, spec.V, spec.J, spec.T, spec.seed)
    buf = torch.full((L * L + 64,), 0x55, dtype=torch.uint8, device="cuda")
    scratch = torch.empty(lat.scratch_bytes(L, 0), dtype=torch.uint8, device="cuda")
    p = lat.LatParams(L=L, encoding=0, n=spec.n, Delta=spec.Delta, V=spec.V, J=spec.J, T=spec.T, seed=spec.seed,
                      n_charged=-1, start_sweep=0, init_codes=None)
    h = ctypes.c_void_p()
    lib = lat.lib()
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.lattice_create(ctypes.byref(p), buf.data_ptr() + 32 + offset, L * L, scratch.data_ptr(),
                              scratch.numel(), stream, ctypes.byref(h)) == 0
    assert lib.lattice_sweep(h, 5) == 0
    torch.cuda.synchronize()
    o.sweeps(5)
    got = buf.cpu().numpy()
    assert np.array_equal(got[32 + offset:32 + offset + L * L].astype(np.int8), o.codes)
    assert (got[:32 + offset] == 0x55).all() and (got[32 + offset + L * L:] == 0x55).all()
    assert lib.lattice_destroy(h) == 0
