"""CDF rows whose F_j = floor(F_max C_j) decreases somewhere: the running maximum has to be taken exactly
there.  Mixtures with one negative weight (C stays in [0, 1]) have such rows; the table must be the running
maximum of the 64-bit F, within the one count of table parity."""
import ctypes

import numpy as np
import pytest
import torch
from scipy.special import ndtr

from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def _mixtures(n, K, nsym, kind, rng):
    """[n][3K]: a rise, a fall, a rise (and with K = 4 a second fall inside the last rise)."""
    c = rng.integers(-nsym // 4, nsym // 4 + 1, n) + (0.5 if kind == "alike" else 0.0)
    if kind == "dips":           # falls over several entries, of a few to thousands of counts
        d, s, fall, fs = rng.uniform(8, 14, n), rng.uniform(1, 2.5, n), rng.choice([3e-3, 0.05, 0.3], n), rng.uniform(0.3, 2, n)
    elif kind == "steps":        # one fall, between two neighbouring entries, anywhere in a wide window
        d, s, fall, fs = rng.uniform(9, 16, n), rng.uniform(0.5, 1.5, n), rng.uniform(0.02, 0.3, n), np.full(n, 0.1)
    else:                        # the same in windows of one length, nine entries
        d, s, fall, fs = np.full(n, 3.0), np.full(n, 0.3), rng.uniform(0.02, 0.3, n), np.full(n, 0.1)
    at = c + 0.5 if kind == "alike" else np.round(c + rng.uniform(-0.4, 0.4, n) * d)
    w = np.stack([np.full(n, 0.6), 0.4 + fall, -fall], 1)
    mu, sg = np.stack([c - d, c + d, at], 1), np.stack([s, s, fs], 1)
    if K == 4:
        w = np.concatenate([w[:, :1], w[:, 1:2] / 2, w[:, 2:], w[:, 1:2] / 2], 1)
        mu, sg = np.concatenate([mu, mu[:, 1:2]], 1), np.concatenate([sg, sg[:, :1]], 1)
    return np.concatenate([w, mu, sg], 1).astype(np.float32)


def _F(prm, K, dist, smin, nsym):
    """F_j, j = 1 .. nsym - 1, before the running maximum (64 bits), and the windows [j1, j2)."""
    p = prm.astype(np.float64)
    w, mu, sg = p[:, :K], p[:, K:2 * K], p[:, 2 * K:]
    j = np.arange(1, nsym)
    z = ((smin + j - 0.5)[None, :, None] - mu[:, None]) / sg[:, None]
    low = ndtr(z) if dist == 0 else np.where(z < 0, 0.5 * np.exp(-abs(z)), 1 - 0.5 * np.exp(-abs(z)))
    up = ndtr(-z) if dist == 0 else np.where(z < 0, 1 - 0.5 * np.exp(-abs(z)), 0.5 * np.exp(-abs(z)))
    S = w.sum(1)[:, None]
    L, U = (w[:, None] * low).sum(2) / S, (w[:, None] * up).sum(2) / S
    fmax = 65536 - nsym
    F = np.where(L <= U, np.floor(fmax * L), fmax - np.maximum(np.ceil(fmax * U), 1)).astype(np.int64)
    tz = np.float32(4.5 if dist == 0 else 11)
    f = prm[:, K:2 * K], prm[:, 2 * K:]
    lo, hi = (f[0] - tz * f[1]).min(1), (f[0] + tz * f[1]).max(1)
    j1 = np.clip(np.floor(lo - smin + np.float32(0.5)) + 1, 1, nsym).astype(np.int64)
    j2 = np.maximum(np.clip(np.ceil(hi - smin + np.float32(0.5)) - 1, 0, nsym - 1).astype(np.int64) + 1, j1)
    F = np.where(j[None] < j1[:, None], 0, np.where(j[None] >= j2[:, None], fmax - 1, F))
    return np.maximum(F, 0), j1, j2


# 16 rows a workgroup up to 40 960 rows, 64 above
@pytest.mark.parametrize("n,rows", [(40000, 16), (98304 + 64 * 400 + 5, 64)])
@pytest.mark.parametrize("kind", ["dips", "steps", "alike"])
@pytest.mark.parametrize("K,dist,smin,smax", [(3, 0, -64, 64), (3, 1, -127, 127), (4, 0, -40, 41)])
def test_running_maximum_where_F_decreases(K, dist, smin, smax, kind, n, rows):
    need_gpu()
    from paper_2405_12631_amd import _lib as L
    say("decreasing F", K, dist, kind, n)
    rng = np.random.default_rng(n + K)
    nsym = smax - smin + 1
    m = min(n, 30000)                       # distinct rows; the launch repeats them
    m -= m % 64
    prm = _mixtures(m, K, nsym, kind, rng)
    F, j1, j2 = _F(prm, K, dist, smin, nsym)
    falls = F[:, 1:] < F[:, :-1]            # column k: entry k + 2 below entry k + 1
    assert falls.any(1).mean() > 0.5
    if dist == 0 and kind != "dips":        # one fall a row, some of them at the first of 64 dealt entries
        assert (falls.sum(1) <= 1).mean() > 0.95
        first = np.concatenate([np.zeros((m // rows, 1), np.int64), np.cumsum((j2 - j1).reshape(-1, rows), 1)], 1)[:, :-1]
        r, k = np.nonzero(falls)
        # (rows of nine entries begin 64 only in the longer workgroup)
        assert ((first.reshape(-1)[r] + k + 2 - j1[r]) % 64 == 0).sum() > 50 or (kind == "alike" and rows == 16)
    if kind == "alike" and dist == 0:
        assert set(j2 - j1) == {9}
    full = torch.from_numpy(prm).cuda().repeat((n + m - 1) // m, 1)[:n].contiguous()
    out = torch.empty((n, nsym + 1), dtype=torch.int16, device="cuda")
    L.call("wv_cdf_tables", full.data_ptr(), n, K, dist, smin, smax, 16, out.data_ptr(),
           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    got = out.cpu().numpy().view(np.uint16).astype(np.int64)
    assert np.array_equal(got[:m], got[m:2 * m][:m] if n >= 2 * m else got[:m]) and not got[:, -1].any()
    ref = np.maximum.accumulate(F, 1) + np.arange(1, nsym)
    assert not got[:m, 0].any() and np.abs(got[:m, 1:-1] - ref).max() <= 1
    assert (np.diff(got[:, :-1], axis=1) >= 1).all()
