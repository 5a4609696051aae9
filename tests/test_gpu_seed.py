"""Initial states seeded on the device: the same codes as the oracle's sort for
every encoding, at the smallest and odd sides, for empty, full and one-signed
charge sets, at any byte address, and where the device hands the work back to the
host.
"""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2301_11735_amd as lat

pytestmark = pytest.mark.gpu


def _same(L, enc, n, n_charged, seed):
    print(f"case seed L={L} enc={enc} n={n} n_charged={n_charged}", flush=True)
    g = lat.Lattice(L, n, 0.1, 0.5, 1.0, 1.0, seed, encoding=enc, n_charged=n_charged)
    o = oracle.OracleLattice(L, n, 0.1, 0.5, 1.0, 1.0, seed, n_charged)
    assert np.array_equal(g.read_state(), o.codes)
    r = g.observables()
    assert r.ints() == o.observables().tolist()
    assert [r.sweep, r.track_nD, r.track_nV, r.track_nJ] == [0, 0, 0, 0]
    g.sweep(2)
    o.sweeps(2)
    assert np.array_equal(g.read_state(), o.codes)


@pytest.mark.parametrize("L,enc", [(28, 0), (32, 0), (36, 0), (64, 1), (100, 0), (320, 0), (448, 1), (1024, 1)])
@pytest.mark.parametrize("n,n_charged", [(0.1, -1), (0.0, 0), (0.0, 2), (-0.4, -1)])
def test_codes_match_oracle(L, enc, n, n_charged):
    _same(L, enc, n, n_charged, 12345678901 + L)


@pytest.mark.parametrize("n", [1.0, -1.0])
def test_every_site_charged(n):
    _same(64, 1, n, 64 * 64, 5)


@pytest.mark.parametrize("candidates", ["0", "1"])
def test_handed_back_to_the_host(candidates, monkeypatch):
    monkeypatch.setenv("LATTICE_SEED_CANDIDATES", candidates)
    for L, enc in ((64, 0), (128, 1)):
        _same(L, enc, 0.2, -1, 99 + L)


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_states_at_any_byte_address(offset):
    import torch

    L = 52
    print(f"case seed at byte offset {offset}", flush=True)
    o = oracle.OracleLattice(L, 0.1, 0.1, 0.5, 1.0, 1.0, 8)
    buf = torch.full((L * L + 64,), 0x55, dtype=torch.uint8, device="cuda")
    scratch = torch.empty(lat.scratch_bytes(L, 0), dtype=torch.uint8, device="cuda")
    p = lat.LatParams(L=L, encoding=0, n=0.1, Delta=0.1, V=0.5, J=1.0, T=1.0, seed=8, n_charged=-1, start_sweep=0,
                      init_codes=None)
    h = ctypes.c_void_p()
    lib = lat.lib()
    assert lib.lattice_create(ctypes.byref(p), buf.data_ptr() + 32 + offset, L * L, scratch.data_ptr(), scratch.numel(),
                              torch.cuda.current_stream().cuda_stream, ctypes.byref(h)) == 0
    got = buf.cpu().numpy()
    assert np.array_equal(got[32 + offset:32 + offset + L * L].astype(np.int8), o.codes)
    assert (got[:32 + offset] == 0x55).all() and (got[32 + offset + L * L:] == 0x55).all()
    assert lib.lattice_destroy(h) == 0
