"""The large-summary selection at the sizes where a unit's rows go to more workgroups: decode over token-major
caches, plain and with append, against the oracle on the list the GPU picked (selections within a 1e-3 band)."""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl
from helpers import assert_attention_close, assert_topk_within_band, to_device_cache
from test_gpu_token_major import decode_and_check, env, say, small  # noqa: F401 (env: the fixture)

pytestmark = pytest.mark.gpu

CASES = [  # units, eight-page runs of the cache, tokens short of the last page's end
    (1, 64, 0), (1, 127, 5), (1, 128, 0), (1, 129, 9), (1, 300, 1), (8, 130, 3), (32, 128, 7), (33, 128, 2), (65, 66, 0),
    (1, 525, 3), (5, 513, 0),  # three workgroups to begin with: twelve
]


@pytest.mark.parametrize("units,runs,short", CASES)
def test_decode(env, oracle, units, runs, short):
    w = small("tiny", batch=units, n_q_heads=2, n_kv_heads=1, context=runs * 16 - short, page_size=2, channel_budget=128,
              token_budget=200, n_heavy=4)
    say("score split", units, runs, short)
    decode_and_check(env, oracle, w, wl.generate(w), 0, None)


@pytest.mark.parametrize("units,runs,short", CASES)
def test_append(env, oracle, units, runs, short):
    """The token goes to the last page, an existing or a new one; every workgroup sees it."""
    torch, rk, dev = env
    n = runs * 16 - short - 1  # tokens before the step
    w = small("tiny", batch=units, n_q_heads=2, n_kv_heads=1, context=n + 1, page_size=2, channel_budget=128,
              token_budget=200, n_heavy=4)
    say("score split append", units, runs, short)
    d = wl.generate(w)
    before = dict(d, K=np.ascontiguousarray(d["K"][:, :, :n]), V=np.ascontiguousarray(d["V"][:, :, :n]),
                  seq_lens=np.full(units, n, dtype=np.int32))
    cache, q = to_device_cache(rk, torch, before, 2, 2, dev, pages_cap=runs * 8, v_layout=rk.V_TOKEN_MAJOR)
    kmax, kmin = rk.alloc_summaries(cache)
    rk.build_page_summaries(cache, kmax, kmin)
    k_new, v_new = (wl.from_bits(np.ascontiguousarray(d[x][:, :, n]), dev) for x in ("K", "V"))
    out = torch.empty((units, 2, 128), dtype=torch.bfloat16, device=dev)
    pages = torch.empty((units, 1, rk.pages_row_len(cache, 200)), dtype=torch.int32, device=dev)
    ws = rk.alloc_workspace(rk.OP_HSA_DECODE, cache, 200)
    rk.hsa_decode_append(cache, q, k_new, v_new, kmax, kmin, 128, 200, 0, out, None, pages, None, ws)
    torch.cuda.synchronize()
    assert cache.seq_lens.cpu().tolist() == [n + 1] * units
    lens = np.full(units, n + 1, dtype=np.int32)
    want_y, _ = oracle.attend_given(d["q"], d["K"], d["V"], lens, 2, pages.cpu().numpy())
    assert_attention_close(wl.to_bits(out), want_y, "y")
    ref = oracle.hsa_decode(d["q"], d["K"], d["V"], lens, 2, 128, 200, want_scores=True)
    P, kp = (n + 2) // 2, oracle.pages_to_pick(n + 1, 2, 200)
    for u in range(units):
        assert_topk_within_band(ref["scores"][u, 0, :P], pages[u, 0].cpu().numpy(), kp, f"unit {u}")
    K2, V2 = rk.unpack_cache(cache)
    assert np.array_equal(wl.to_bits(K2)[:, :, :n + 1], d["K"]) and np.array_equal(wl.to_bits(V2)[:, :, :n + 1], d["V"])
    bounds = oracle.build_summaries(d["K"], lens, 2, cache.pages_cap)
    for got, want in zip((kmax, kmin), bounds):
        ok = ~np.isnan(want)
        assert np.array_equal(wl.bf16_bits_to_f64(wl.to_bits(got))[ok], want[ok])
