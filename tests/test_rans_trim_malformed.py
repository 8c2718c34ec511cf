"""The host coder on trimmed rows that no wv_cdf_trim makes (F falls somewhere, or lies above the plateau): a
stream that the full tables decode is decoded, to the same symbols, and nothing else than a status comes
of the rest."""
import ctypes

import numpy as np

from paper_2405_12631_amd import _lib as L


def test_no_stream_is_refused_that_the_full_tables_decode():
    rng = np.random.default_rng(0)
    lib, accepted, statuses = L.lib(), 0, set()
    for _ in range(4000):
        nsym, n = int(rng.choice([2, 3, 7, 42, 129, 255])), int(rng.integers(1, 30))
        lolen, packed = np.empty((n, 2), np.uint8), []
        for i in range(n):
            lo = int(rng.integers(1, nsym + 1))
            ln = int(rng.integers(0, nsym - lo + 1))
            f = rng.integers(0, 65536 if rng.random() < 0.3 else 65535 - nsym, ln)
            f = np.sort(f) if rng.random() < 0.7 else f
            if ln and rng.random() < 0.3:
                f[rng.integers(0, ln)] = rng.integers(0, 65536)
            lolen[i] = lo, ln
            packed.append(f)
        pk = np.concatenate(packed + [np.zeros(0)]).astype(np.uint16)
        buf = pk if pk.size else np.zeros(1, np.uint16)
        full = np.empty((n, nsym + 1), np.uint16)
        L.call("wv_cdf_untrim", lolen.ctypes.data, buf.ctypes.data, pk.size, nsym, n, full.ctypes.data)
        sym = rng.integers(0, nsym, n).astype(np.uint8)
        out, ln = np.zeros(16 + 4 * n, np.uint8), ctypes.c_size_t()
        rc = lib.wv_rans_encode_trim(lolen.ctypes.data, buf.ctypes.data, pk.size, nsym, sym.ctypes.data, n,
                                     out.ctypes.data, out.size, ctypes.byref(ln))
        streams = [rng.integers(0, 256, 40 + 4 * n).astype(np.uint8)] + ([out[:ln.value].copy()] if rc == 0 else [])
        for data in streams:
            a, b = np.zeros(n, np.uint8), np.zeros(n, np.uint8)
            ra = lib.wv_rans_decode(full.ctypes.data, nsym, n, data.ctypes.data, data.size, a.ctypes.data)
            rb = lib.wv_rans_decode_trim(lolen.ctypes.data, buf.ctypes.data, pk.size, nsym, n, data.ctypes.data,
                                         data.size, b.ctypes.data)
            statuses |= {ra, rb}
            if ra == 0:
                accepted += 1
                assert rb == 0 and np.array_equal(a, b)
    assert accepted > 2000 and statuses == {L.WV_OK, L.WV_ECORRUPT}
