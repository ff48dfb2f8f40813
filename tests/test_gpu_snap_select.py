"""Stage 1's max-pool and select at the edges of their tiles: pooling widths around the groups of eight,
prompts that end inside a group, tile or slice, the three sizes of run list a workgroup handles, votes
with so many ties that one pass of bins cannot decide, and a wanted vote at the upper end of the lowest bin.

Selections: exact outside a 1e-3 band around the threshold (the GPU sums votes in fp32, the oracle in fp64);
where every vote is one of a few well separated values, exact with the tie rule."""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl
from helpers import assert_topk_within_band, to_device_cache

pytestmark = pytest.mark.gpu
W = 16


def kept_of(oracle, d, hq, ks, keep):
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    dev = torch.device("cuda:0")
    B, hkv = d["K"].shape[:2]
    src, _ = to_device_cache(rk, torch, d, hq, 16, dev)
    dst = rk.alloc_cache(B, hq, hkv, 128, 16, (keep + 15) // 16, dev, zero=True)
    kept = torch.full((B, hkv, keep), -9, dtype=torch.int32, device=dev)
    ws = rk.alloc_workspace(rk.OP_SNAPKV, src, W, keep)
    ws.fill_(0xEE)
    rk.workspace_init(ws)
    for _ in range(2):  # the second call finds the run counts of the first
        rk.snapkv_compress(wl.from_bits(d["qobs"], dev), src, W, ks, keep, dst, kept, ws)
        torch.cuda.synchronize()
    return kept.cpu().numpy(), oracle.snapkv(d["qobs"], d["K"], d["seq_lens"], ks, keep, want_votes=True)


def draw(lens, hkv, seed=1):
    w = wl.scaled(wl.CONFIGS["tiny"], batch=len(lens), n_q_heads=hkv, n_kv_heads=hkv, context=max(lens), window=W,
                  n_heavy=4, seed=seed)
    d = wl.generate(w, with_obs=True)
    d["seq_lens"] = np.asarray(lens, dtype=np.int32)
    return d


@pytest.mark.parametrize("ks", [1, 3, 13, 15, 17, 23, 31, 33, 63, 1023])
@pytest.mark.parametrize("lens,keep", [((1000, 333), 77), ((4096 + W + 5, 1024 + W), 300), ((9001, 8192 + W), 64)])
def test_pool_widths(oracle, ks, lens, keep):
    print("[case] pool", ks, lens, keep, flush=True)
    d = draw(lens, 2)
    got, ref = kept_of(oracle, d, 2, ks, keep)
    for b, S in enumerate(lens):
        for g in range(2):
            assert got[b, g, keep - W:].tolist() == list(range(S - W, S))
            assert_topk_within_band(ref["pooled"][b, g, :S - W], got[b, g, :keep - W], keep - W, f"b{b} g{g}")


@pytest.mark.parametrize("S", [8192 + W, 8200 + W, 20000, 24576 + W, 33001])
def test_list_sizes(oracle, S):
    """Unpooled votes: as many runs as positions, around what a workgroup keeps in registers and beyond."""
    print("[case] runs", S, flush=True)
    d = draw((S,), 1)
    got, ref = kept_of(oracle, d, 1, 1, 513)
    assert_topk_within_band(ref["pooled"][0, 0, :S - W], got[0, 0, :513 - W], 513 - W, "kept")


@pytest.mark.parametrize("values", [1, 5, 9])
@pytest.mark.parametrize("S,keep,ks", [(5000, 1111, 1), (30000, 700, 1), (30000, 3000, 7)])
def test_ties(oracle, values, S, keep, ks):
    """Every key is one of `values` rows, so votes repeat exactly: ties go to the lower position."""
    print("[case] ties", values, S, keep, ks, flush=True)
    d = draw((S,), 1, seed=3)
    rng = np.random.default_rng(S + values)
    d["K"] = np.ascontiguousarray(d["K"][:, :, rng.integers(0, values, size=S)])
    got, ref = kept_of(oracle, d, 1, ks, keep)
    assert got[0, 0].tolist() == ref["kept"][0, 0].tolist()


@pytest.mark.parametrize("S,ks,share", [(5000, 1, 0.5), (5000, 1, 0.0), (20000, 1, 0.9), (5000, 3, 0.5)])
def test_lowest_bin(oracle, S, ks, share):
    """One token takes nearly all the weight; the other votes lie around 2^-56, where the lowest bin ends, in levels
    1/64 octave apart or more.  The wanted one is the highest level of that bin, with more smaller votes in
    the bin than are ranked at once and others just above it.  Votes in fp32 are off by 1e-5 or so, the levels
    by 1e-2: exact."""
    print("[case] lowest bin", S, ks, share, flush=True)
    rng = np.random.default_rng(S + ks)
    wanted = 1 + 1 / 128
    levels = np.array([2.0**-5, 2.0**-3, 2.0**-2, 0.5, 0.75, wanted] + [wanted + i / 64 for i in range(1, 8)])
    f = rng.choice(levels, size=S, p=[0.1] * 5 + [0.08] + [0.06] * 7)
    f[S - W:] = levels[0]
    # q . k / sqrt(128) = log(f) - 60 log 2: a vote is W of those probabilities
    coarse, q0 = -58.75, 8.0
    k1 = (np.log(f) - 60 * np.log(2.0)) * np.sqrt(128.0) - coarse * q0
    K = np.zeros((1, 1, S, 128), dtype=np.float32)
    K[0, 0, :, 0], K[0, 0, :, 1] = coarse, k1
    heavy = 4321 % (S - W)
    K[0, 0, heavy] = 0.0
    qobs = np.zeros((1, 1, W, 128), dtype=np.float32)
    qobs[..., 0], qobs[..., 1] = q0, 1.0
    f[heavy] = 2.0**56
    r = ks // 2
    pooled = np.array([f[max(0, j - r):min(S - W, j + r + 1)].max() for j in range(S - W)])
    above, at = int((pooled > wanted).sum()), int((pooled == wanted).sum())
    assert (pooled <= wanted).sum() > 512 and at > 2
    keep = W + above + max(1, int(share * at))
    d = dict(qobs=wl.f32_to_bf16_bits(qobs), K=wl.f32_to_bf16_bits(K), V=wl.f32_to_bf16_bits(K),
             q=wl.f32_to_bf16_bits(qobs[:, :, 0]), seq_lens=np.array([S], dtype=np.int32))
    got, ref = kept_of(oracle, d, 1, ks, keep)
    theta = np.sort(ref["pooled"][0, 0, :S - W])[::-1][keep - W - 1]
    assert 2.0**-56 * (1 + 1e-3) < theta < 2.0**-56 * (1 + 1 / 64 - 1e-3)
    assert got[0, 0].tolist() == ref["kept"][0, 0].tolist()
