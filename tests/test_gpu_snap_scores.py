"""Stage 1's score passes at the edges of their tiles: blocks of 32 softmax rows that are real in part, one and two
column groups, windows that do not divide a block, prompts that end inside a page, pair, segment and chunk, and the
longest chunk (whose size follows from the capacity: the table is padded with absent pages).

Kept positions against the oracle on unpooled votes, exact outside a 1e-3 band around the threshold (votes are sums of
at most 256 probabilities, whose logits are summed in fp32: some 1e-6 relative)."""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl
from helpers import assert_topk_within_band, to_device_cache

pytestmark = pytest.mark.gpu


def check(oracle, hq, hkv, W, lens, cap, keep):
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    print("[case] scores", hq, hkv, W, lens, cap, keep, flush=True)
    dev = torch.device("cuda:0")
    w = wl.scaled(wl.CONFIGS["tiny"], batch=len(lens), n_q_heads=hq, n_kv_heads=hkv, context=max(lens), window=W, n_heavy=4,
                  seed=hq * 100 + W)
    d = wl.generate(w, with_obs=True)
    d["seq_lens"] = np.asarray(lens, dtype=np.int32)
    src, _ = to_device_cache(rk, torch, d, hq, 16, dev, shuffle_rng=np.random.default_rng(W))
    held = src.block_table
    src.pages_cap = max(cap, held.shape[1])
    src.block_table = torch.full((len(lens), src.pages_cap), -1, dtype=torch.int32, device=dev)
    src.block_table[:, :held.shape[1]] = held
    dst = rk.alloc_cache(len(lens), hq, hkv, 128, 16, (keep + 15) // 16, dev, zero=True)
    kept = torch.full((len(lens), hkv, keep), -9, dtype=torch.int32, device=dev)
    size = rk.workspace_bytes(rk.OP_SNAPKV, src, W, keep)
    ws = torch.full((size + 4096,), 0xCD, dtype=torch.uint8, device=dev)  # what lies behind the workspace stays as it is
    rk.snapkv_compress(wl.from_bits(d["qobs"], dev), src, W, 1, keep, dst, kept, ws[:size])
    torch.cuda.synchronize()
    assert (ws[size:] == 0xCD).all()
    got, ref = kept.cpu().numpy(), oracle.snapkv(d["qobs"], d["K"], d["seq_lens"], 1, keep, want_votes=True)
    for b, S in enumerate(lens):
        for g in range(hkv):
            assert got[b, g, keep - W:].tolist() == list(range(S - W, S))
            assert_topk_within_band(ref["gv"][b, g, :S - W], got[b, g, :keep - W], keep - W, f"b{b} g{g}")


# softmax rows (group x window): 16, 32, 48, 64 | 80, 96, 128 | 144, 192, 256 in two column groups
@pytest.mark.parametrize("hq,hkv,W", [(1, 1, 16), (2, 1, 16), (3, 1, 16), (8, 2, 16), (5, 1, 16), (2, 1, 48), (4, 1, 32),
                                      (3, 1, 48), (4, 1, 48), (8, 1, 32), (2, 1, 128)])
def test_rows(oracle, hq, hkv, W):
    check(oracle, hq, hkv, W, (1500, 512 + W, 1024 + W + 16, 700 + W), 0, 200)


@pytest.mark.parametrize("hq,hkv,W", [(4, 4, 16), (16, 4, 16), (64, 4, 16)])
@pytest.mark.parametrize("last", [0, 1, 15, 16, 17, 32, 255, 1024, 1039])
def test_chunk_ends(oracle, hq, hkv, W, last):
    """Chunks of the longest kind (128 pages) and what lies behind them."""
    check(oracle, hq, hkv, W, (8192 + W + last, 4096 + W + last, 2000 + last, 8192 + last), 8448, 300)


@pytest.mark.parametrize("hq,hkv,W", [(2, 2, 16), (16, 2, 16), (4, 1, 32)])
@pytest.mark.parametrize("cap,chunk", [(512, 8), (520, 16), (1024, 16), (1032, 32)])
def test_short_chunks(oracle, hq, hkv, W, cap, chunk):
    """Capacities at which four units' workgroups are just as many as compute units, and the next longer ones."""
    t = 16 * chunk  # tokens a workgroup scores
    check(oracle, hq, hkv, W, tuple(x + W for x in (3 * t, 3 * t + 1, 5 * t - 1, 4 * t + 17))[:4 // hkv], cap, 200)


@pytest.mark.parametrize("hq,cap", [(64, 2560), (16, 2304), (32, 6400), (32, 8192), (32, 8320), (16, 8320)])
def test_merged_statistics(oracle, hq, cap):
    """Chunks of 128 pages in sixteen units: more of them than a thread of the second pass merges at a time (20 of 256 softmax
    rows, 50 of 128), 18 of 64 rows dealt to four threads, as many statistics and workgroups as it merges at most (64 of 128
    rows), one chunk more, and one more with fewer rows."""
    check(oracle, hq, 4, 16, (33000, 2064, 18 * 2048 + 16 if cap == 2304 else 20 * 2048, 300), cap, 200)


@pytest.mark.parametrize("hkv,lens,cap", [(2, (4096, 4000, 1500, 2100), 256), (1, (32768,), 2048)])
def test_most_chunk_statistics(oracle, hkv, lens, cap):
    """256 softmax rows in 256 workgroups of 8 pages, whose statistics take more room than the buffers they share; merged by the
    second pass (eight units) and by a launch (one unit)."""
    check(oracle, hkv * 8, hkv, 32, lens, cap, 100)
