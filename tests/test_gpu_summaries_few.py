"""Page summaries of few pages, which go to workgroups of 16 pages: exact against the oracle's bounds."""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl
from helpers import to_device_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,ctx,ps,first,count", [
    (1, 255, 16, 0, -1), (1, 257, 16, 3, 9), (2, 1000, 4, 0, -1), (2, 777, 5, 1, 100), (1, 4099, 64, 0, -1), (1, 100, 1, 7, 33)])
def test_summaries_of_few_pages(oracle, B, ctx, ps, first, count):
    """Bounds equal the oracle's in the range asked for; nothing else is written."""
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    print("[case] summaries", B, ctx, ps, first, count, flush=True)
    d = wl.generate(wl.scaled(wl.CONFIGS["tiny"], batch=B, context=ctx, page_size=ps))
    cache, _ = to_device_cache(rk, torch, d, 16, ps, torch.device("cuda:0"), v_layout=0 if ps == 16 else 1)
    kmax, kmin = rk.alloc_summaries(cache)
    kmax.fill_(7.0), kmin.fill_(7.0)
    rk.build_page_summaries(cache, kmax, kmin, first, count)
    torch.cuda.synchronize()
    P = (ctx + ps - 1) // ps
    last = P if count < 0 else min(P, first + count)
    want = oracle.build_summaries(d["K"], d["seq_lens"], ps, cache.pages_cap)
    for got, w in zip((kmax, kmin), want):
        bits = wl.to_bits(got)
        assert np.array_equal(wl.bf16_bits_to_f64(bits)[..., first:last], w[..., first:last])
        assert (bits[..., :first] == 0x40E0).all() and (bits[..., last:] == 0x40E0).all()
