"""The C ABI library loads on the CPU and exports every symbol the header
declares; host-only entry points behave as documented (no GPU calls)."""
import ctypes
import re
import os

import pytest

import paper_2305_07545_amd as P
from paper_2305_07545_amd import kmerco

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "kmerco.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kc_[a-z_]+)\s*\(", text)))


def test_header_declares_the_abi():
    names = declared_functions()
    assert "kc_insert" in names and "kc_classify" in names and "kc_create" in names


def test_library_exports_every_declared_symbol():
    lib = P.load_library()
    for name in declared_functions():
        assert hasattr(lib, name), name
    assert set(declared_functions()) == set(kmerco.SIGNATURES)


def test_dims_matches_oracle(oracle_lib):
    for n in [1, 10, 1000, 5.5e5, 6.1e7, 20484059 / 2, 163872472 / 2, 8.9e9]:
        assert P.dims(n) == oracle_lib.dims(n)


def test_dims_errors():
    for bad in [(0, 0.001), (10, 0.0), (10, 1.0), (-1, 0.5)]:
        with pytest.raises(P.KmercoError):
            P.dims(*bad)


def test_eta_and_strings():
    assert [P.eta(a) for a in (1, 5, 8, 16, 32, 64, 0, 65)] == [64, 12, 8, 4, 2, 1, 0, 0]
    assert P.strerror(0) == "ok"
    assert "capacity" in P.strerror(-3)
    assert P.load_library().kc_version() >= 1


def test_create_rejects_bad_layouts_without_touching_the_device():
    lib = P.load_library()
    h = ctypes.c_void_p(None)
    bad = [(0, 5, 8, 1), (5, 0, 8, 1), (5, 7, 0, 1), (5, 7, 33, 1), (5, 7, 8, 0), (5, 7, 8, 9)]
    for X, Y, a, kh in bad:
        L = kmerco.kc_layout(X, Y, a, kh)
        st = lib.kc_create(ctypes.byref(L), ctypes.c_void_p(0x1000), 1, None, ctypes.byref(h))
        assert st == kmerco.KC_EINVAL
    L = kmerco.kc_layout(5, 7, 8, 1)
    assert lib.kc_create(ctypes.byref(L), None, 1, None, ctypes.byref(h)) == kmerco.KC_EINVAL


def test_null_handle_calls_are_rejected():
    lib = P.load_library()
    assert lib.kc_insert(None, None, None, 0, 0, 21, None, 0, None, None, None) == kmerco.KC_EINVAL
    assert lib.kc_classify(None, None, None, 0, 2, None, None, None, None, None) == kmerco.KC_EINVAL
    assert lib.kc_query(None, None, 0, None, None) == kmerco.KC_EINVAL
    assert lib.kc_sync(None) == kmerco.KC_EINVAL
    assert lib.kc_reserve(None, 10) == kmerco.KC_EINVAL
    lib.kc_destroy(None)


def test_filter_and_scratch_bytes_on_the_host():
    """kc_filter_bytes is X*Y*8; kc_scratch_bytes counts what kc_reserve would
    allocate without a device: about 22 bytes per base on the single-level
    binned path (a 150 M-base insert into the 55.7 MB countBF), growing with
    the reservation and with the hash functions, 0 for invalid layouts."""
    assert P.filter_bytes(2621, 2657) == 2621 * 2657 * 8
    assert P.filter_bytes(0, 5) == 0 and P.scratch_bytes(5, 7, 100, alpha=0) == 0
    sizes = [P.scratch_bytes(2621, 2657, n) for n in (0, 1000, 10**6, 150 * 10**6, 2**28)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:])) and sizes[0] > 0
    per_base = sizes[3] / (150 * 10**6)
    assert 20 < per_base < 25, per_base
    assert P.scratch_bytes(2621, 2657, 10**7, k_h=3) > P.scratch_bytes(2621, 2657, 10**7)
    # beyond one chunk of the binned path the per-chunk scratch stops growing
    assert P.scratch_bytes(2621, 2657, 2**30) - P.scratch_bytes(2621, 2657, 2**29) < \
        12 * 2**29


def test_scratch_bytes_rounds_every_piece():
    """Every piece kc_scratch_bytes counts is rounded up to 256 bytes (the
    carving of a caller's scratch lays them out at that alignment), and the
    partitioned path's need per base (about 19 bytes) is below the
    single-level path's (about 22).  An insert of several chunks also holds
    the carried first-seen records: 6 bytes per position before the last
    chunk."""
    for X, Y, n in [(269, 281, 10**6), (2621, 2657, 10**7), (31627, 31657, 10**8)]:
        assert P.scratch_bytes(X, Y, n) % 256 == 0
    one_chunk = 2**32 - 2**16  # the partitioned path's chunk
    big = P.scratch_bytes(31627, 31657, one_chunk) / one_chunk
    assert 15 < big < 22, big

    def second_chunk(**kw):  # bytes per base the second chunk adds
        return (P.scratch_bytes(31627, 31657, 2 * one_chunk, **kw) -
                P.scratch_bytes(31627, 31657, one_chunk, **kw)) / one_chunk

    # eta = 4 (alpha = 16) and two hash functions carry nothing: the per-
    # position buffers only; eta = 8 adds the 6-byte records
    assert 1 < second_chunk(alpha=16) < 3 and 1 < second_chunk(k_h=2) < 3
    assert 5.99 < second_chunk() - second_chunk(alpha=16) < 6.01


def test_create_in_rejects_bad_arguments_on_the_host():
    """k above 64 and a misaligned scratch buffer are refused before any
    device call."""
    lib = P.load_library()
    h = ctypes.c_void_p(None)
    L = kmerco.kc_layout(5, 7, 8, 1)
    w = ctypes.c_void_p(0x1000)
    assert lib.kc_create_in(ctypes.byref(L), w, 0, 65, None, 0, 0, None,
                            ctypes.byref(h)) == kmerco.KC_EINVAL
    assert lib.kc_create_in(ctypes.byref(L), w, 1, 0, ctypes.c_void_p(0x1010), 1 << 20, 0, None,
                            ctypes.byref(h)) == kmerco.KC_EINVAL


def test_winner_records_turned_off_bound_the_chunk(monkeypatch):
    """KMERCO_WINNER_RECORDS=0: partitioned chunks are small enough for the
    region pass to sort its records itself, 2^28 positions."""
    def scratch():
        return P.scratch_bytes(31627, 31657, 2**30)
    one_chunk = scratch()
    monkeypatch.setenv("KMERCO_WINNER_RECORDS", "0")
    off = scratch()
    monkeypatch.delenv("KMERCO_WINNER_RECORDS")
    monkeypatch.setenv("KMERCO_CHUNK_POSITIONS", str(2**28))
    assert off == scratch() != one_chunk
