"""The host coder on trimmed rows against the coder on the rebuilt tables: windows of every
length and place, every symbol, and streams cut short."""
import ctypes

import numpy as np
import pytest

from paper_2405_12631_amd import _lib as L


def _rows(rng, n, nsym):
    """Random valid tables and their trimmed form (F non-decreasing, 0 below the window, F_max - 1
    above it, strictly between inside)."""
    top = 65536 - nsym - 1
    lolen, packed, full = np.empty((n, 2), np.uint8), [], np.empty((n, nsym + 1), np.uint16)
    for i in range(n):
        lo = int(rng.integers(1, nsym + 1))
        ln = int(rng.choice([0, 1, 2, 3, nsym - lo, rng.integers(0, nsym - lo + 1)]))
        ln = min(ln, nsym - lo)
        f = np.sort(rng.integers(1, rng.choice([4, 300, top]), ln))
        F = np.concatenate([np.zeros(lo, np.int64), f, np.full(nsym - lo - ln, top)])
        full[i, :nsym] = np.arange(nsym) + F
        full[i, nsym] = 0
        lolen[i] = lo, ln
        packed.append(f)
    return lolen, np.concatenate(packed + [np.zeros(0)]).astype(np.uint16), full


@pytest.mark.parametrize("nsym", [2, 3, 42, 129, 255])
def test_trimmed_coder_equals_full_table_coder(nsym):
    rng = np.random.default_rng(nsym)
    n = 6 * nsym + 500
    lolen, packed, full = _rows(rng, n, nsym)
    pk = packed if packed.size else np.zeros(1, np.uint16)
    un = np.empty_like(full)
    L.call("wv_cdf_untrim", lolen.ctypes.data, pk.ctypes.data, packed.size, nsym, n, un.ctypes.data)
    assert np.array_equal(un, full)
    for sym in (np.resize(np.arange(nsym), n).astype(np.uint8), rng.integers(0, nsym, n).astype(np.uint8),
                np.zeros(n, np.uint8), np.full(n, nsym - 1, np.uint8)):
        out = [np.empty(16 + 4 * n, np.uint8) for _ in range(2)]
        ln = [ctypes.c_size_t(), ctypes.c_size_t()]
        L.call("wv_rans_encode", full.ctypes.data, nsym, sym.ctypes.data, n, out[0].ctypes.data, out[0].size,
               ctypes.byref(ln[0]))
        L.call("wv_rans_encode_trim", lolen.ctypes.data, pk.ctypes.data, packed.size, nsym, sym.ctypes.data, n,
               out[1].ctypes.data, out[1].size, ctypes.byref(ln[1]))
        a, b = (o[:k.value].tobytes() for o, k in zip(out, ln))
        assert a == b
        for data in (a, a[:-1], a[:len(a) // 2], a[:3], bytes(len(a)), a[:5] + bytes([a[5] ^ 0x55]) + a[6:]):
            src = np.frombuffer(data, np.uint8)
            got = [np.zeros(n, np.uint8) for _ in range(2)]
            rc0 = L.lib().wv_rans_decode(full.ctypes.data, nsym, n, src.ctypes.data, len(data), got[0].ctypes.data)
            rc1 = L.lib().wv_rans_decode_trim(lolen.ctypes.data, pk.ctypes.data, packed.size, nsym, n,
                                              src.ctypes.data, len(data), got[1].ctypes.data)
            assert rc0 == rc1 and np.array_equal(got[0], got[1])
            if data == a:
                assert rc0 == 0 and np.array_equal(got[0], sym)
