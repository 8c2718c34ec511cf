"""CDF rows whose windows hold no entry at all, one, or the same few in every row: the fill of entries in
pairs, and the deal without a search where the windows of a workgroup are of one length."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_common import check_cdf_rows, need_gpu, say
from wvgen import get_config

pytestmark = pytest.mark.gpu


# rows of 130 (even), 43 (odd), 255 (odd) and 42 entries; 16 rows a workgroup, 64, and 64 with a short last one
@pytest.mark.parametrize("n", [1007, 41024, 50001])
@pytest.mark.parametrize("K,dist,smin,smax", [(1, 0, -64, 64), (2, 0, -20, 21), (1, 1, -127, 126), (3, 0, -20, 20)])
def test_narrow_windows_anywhere(K, dist, smin, smax, n):
    need_gpu()
    from paper_2405_12631_amd import _lib as L
    say("narrow windows", K, dist, smin, smax, n)
    nsym = smax - smin + 1
    rng = np.random.default_rng(n + nsym)
    # the window of a component is 9 (Laplace: 22) scales wide: below one entry, about one, about six; per
    # block of 1024 rows, so that whole workgroups are alike; means at every distance from the boundaries,
    # and beyond the alphabet
    width = np.repeat(rng.choice([0.2, 0.9, 5.6], n // 1024 + 1), 1024)[:n]
    sg = np.repeat((width / (22 if dist else 9))[:, None], K, 1)
    mu = np.repeat(np.round(rng.uniform(smin - 4, smax + 4, n) * 64)[:, None] / 64, K, 1)
    prm = np.concatenate([np.full((n, K), 1 / K), mu, sg], 1).astype(np.float32)
    E = nsym + 1
    out = torch.zeros(n * E + 16, dtype=torch.int16, device="cuda")
    d = torch.from_numpy(prm).cuda()
    L.call("wv_cdf_tables", d.data_ptr(), n, K, dist, smin, smax, 16, out.data_ptr(),
           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    got = out.cpu().numpy().view(np.uint16)
    assert not got[n * E:].any()
    cfg = get_config("gray64", mix_k=K, dist="laplace" if dist else "gauss", sym_min=smin, sym_max=smax)
    check_cdf_rows(got[:n * E].reshape(n, E), prm, cfg)
