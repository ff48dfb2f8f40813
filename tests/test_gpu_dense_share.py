"""The Full-KV baseline divides the pages the sequences hold between its workgroups (dense_share in
attend_core.h): one sequence, unequal, empty and over-long ones, fewer and more units than workgroups fit
the chip at once, shares of one, two and four rounds, more than 64 sequences, against the fp64 oracle.

Bar: 1e-2 absolute / relative (bf16 operands and weights, fp32 sums, bf16 results)."""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl
from helpers import assert_attention_close, to_device_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,lens,ps,layout", [
    (4, 1, (1,), 16, 0),                                   # below the line: divided by capacity
    (4, 1, (255, 256, 257), 16, 0),                        # the same, around the smallest share of eight wavefronts
    (32, 8, (9000,), 16, 0),                               # one sequence, in scalar arithmetic
    (32, 8, (9001,), 16, 1),
    (8, 8, (6001,), 3, 1),                                 # below the line
    (32, 8, (0, 5000, 17, 1), 16, 0),                      # an empty sequence among unequal ones
    (15, 5, (3001, 150, 1600, 3100), 16, 0),                     # heads that do not divide the workgroups
    (16, 16, tuple(5 + 47 * i for i in range(20)), 16, 0),  # more units than compute units
    (16, 16, tuple((331 * i) % 820 for i in range(40)), 16, 0),  # more sequences than workgroups of a round; one empty
    (16, 16, tuple((331 * i) % 820 for i in range(40)), 16, 1),
    (8, 8, (3000,) + (40,) * 30, 16, 0),                   # nearly as many, one of them long: more shares than one round holds
    (8, 8, (3900,) * 17, 16, 0),                           # two rounds
    (8, 8, (6400,) * 33, 16, 0),                           # four rounds
    (1, 1, (700,) * 128, 16, 0),                           # the largest batch that is divided: below the line by its rows
    (2, 2, tuple(1600 + i for i in range(128)), 16, 1),    # the largest batch that is divided
    (2, 2, tuple((97 * i) % 1700 for i in range(70)), 16, 0),  # a second block of 64 sequences
    (16, 1, (20000, 31, 9000), 16, 0),                            # the largest group: four wavefronts
    (8, 2, (40000, 700), 16, 0),
    (8, 2, (30000, 0, 333), 3, 1),                          # token-major, pages that do not divide 16
    (32, 8, (2700, 16, 1111), 16, 1),
    (6, 6, tuple(5 + 60 * i for i in range(20)), 1, 1),
    (4, 1, (300, 17), 16, 0),                              # below the line
])
def test_unequal_lengths(oracle, hq, hkv, lens, ps, layout):
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    print("[case] dense share", hq, hkv, lens, ps, layout, flush=True)
    dev = torch.device("cuda:0")
    w = wl.scaled(wl.CONFIGS["tiny"], batch=len(lens), n_q_heads=hq, n_kv_heads=hkv, context=max(lens), page_size=ps,
                  n_heavy=0)
    d = wl.generate(w)
    d["seq_lens"] = np.asarray(lens, dtype=np.int32)
    cache, q = to_device_cache(rk, torch, d, hq, ps, dev, shuffle_rng=np.random.default_rng(5), extra_pages=3,
                               v_layout=layout)
    out = torch.full((len(lens), hq, 128), 7.0, dtype=torch.bfloat16, device=dev)
    lse = torch.full((len(lens), hq), 7.0, dtype=torch.float32, device=dev)
    ws = rk.alloc_workspace(rk.OP_DENSE_DECODE, cache)
    want_y, want_lse = oracle.dense_decode(d["q"], d["K"], d["V"], d["seq_lens"])
    for _ in range(2):  # the second call finds the counters as the first one left them
        rk.dense_decode(cache, q, out, lse, ws)
        torch.cuda.synchronize()
        assert_attention_close(wl.to_bits(out), want_y, "dense y")
        np.testing.assert_allclose(lse.cpu().numpy(), want_lse, rtol=1e-3, atol=1e-3)


@pytest.mark.parametrize("layout", [0, 1])
def test_length_beyond_the_capacity(oracle, layout):
    """A length that exceeds the cache counts as a full one."""
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    print("[case] dense share beyond", layout, flush=True)
    dev = torch.device("cuda:0")
    lens = (2048, 3072, 100)
    d = wl.generate(wl.scaled(wl.CONFIGS["tiny"], batch=3, n_q_heads=32, n_kv_heads=8, context=3072, page_size=16, n_heavy=0))
    d["seq_lens"] = np.asarray(lens, dtype=np.int32)
    cache, q = to_device_cache(rk, torch, d, 32, 16, dev, v_layout=layout)
    assert cache.pages_cap * 16 == 3072
    cache.seq_lens[1] = 3072 + 5000
    out = torch.full((3, 32, 128), 7.0, dtype=torch.bfloat16, device=dev)
    ws = rk.alloc_workspace(rk.OP_DENSE_DECODE, cache)
    want_y, _ = oracle.dense_decode(d["q"], d["K"], d["V"], d["seq_lens"])
    rk.dense_decode(cache, q, out, None, ws)
    torch.cuda.synchronize()
    assert_attention_close(wl.to_bits(out), want_y, "dense y")
