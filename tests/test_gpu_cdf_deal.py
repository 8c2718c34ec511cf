"""CDF tables built from evenly dealt window entries: both workgroup forms and every launch size
give the same rows, at any alignment of the table, and the rows are the oracle's."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_common import check_cdf_rows, need_gpu, say
from wvgen import get_config

pytestmark = pytest.mark.gpu


def _tables(prm, K, dist, smin, smax, offset=0):
    from paper_2405_12631_amd import _lib as L
    n, E = prm.shape[0], smax - smin + 2
    out = torch.zeros(n * E + 8, dtype=torch.int16, device="cuda")
    L.call("wv_cdf_tables", prm.data_ptr(), n, K, dist, smin, smax, 16, out.data_ptr() + 2 * offset,
           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert not out[:offset].any() and not out[offset + n * E:].any()
    return out[offset:offset + n * E].view(n, E)


# 98 304 rows is the last launch of 16-row workgroups; alphabets with even and odd row lengths,
# rows of one, two and a few more than two 64-pair passes.
@pytest.mark.parametrize("K,dist,smin,smax", [(3, 0, -64, 64), (1, 1, -64, 64), (4, 0, -20, 21), (2, 1, -127, 127)])
def test_tables_do_not_depend_on_launch_size_or_alignment(K, dist, smin, smax):
    need_gpu()
    say("cdf deal", K, dist, smin, smax)
    g = torch.Generator(device="cuda").manual_seed(K)
    n = 98304 + 65
    w = torch.softmax(2 * torch.randn(n, K, generator=g, device="cuda"), 1)
    mu = torch.randn(n, K, generator=g, device="cuda") * torch.exp(2 * torch.randn(n, 1, generator=g, device="cuda"))
    sig = torch.exp(1.5 * torch.randn(n, K, generator=g, device="cuda")).clamp_min(0.11)
    # every fourth row: narrow far modes, between which C is flat and its rounding may decrease
    sig[::4] = 0.2 + 2 * torch.rand(sig[::4].shape, generator=g, device="cuda")
    mu[::4] = (torch.rand(mu[::4].shape, generator=g, device="cuda") - 0.5) * 1.2 * (smax - smin)
    prm = torch.cat((w, mu, sig), 1).float().contiguous()
    big = _tables(prm, K, dist, smin, smax)
    for m in (1, 15, 16, 17, 63, 65, 98304):
        assert torch.equal(_tables(prm[:m], K, dist, smin, smax), big[:m]), m
    for off in (1, 2, 3):
        assert torch.equal(_tables(prm, K, dist, smin, smax, off), big), off
        assert torch.equal(_tables(prm[:200], K, dist, smin, smax, off), big[:200]), off
    u = big[:, :-1].to(torch.int32) & 0xFFFF
    assert bool((u[:, 1:] > u[:, :-1]).all()) and not bool(big[:, -1].any())
    cfg = get_config("gray64", mix_k=K, dist="laplace" if dist else "gauss", sym_min=smin, sym_max=smax)
    check_cdf_rows(big[:2000].cpu().numpy().view(np.uint16), prm[:2000].cpu().numpy(), cfg)
