"""The page that receives a token is scored like any other: a fused step picks what append_kv followed by hsa_decode
picks, also where nothing forces the newest page in and its score equals another page's at the threshold.

Per (sequence, KV head): six pages score far above the rest, one early page holds copies of a single key, and the tail
page is filled with that same key, token by token.  Both pages then have the same bounds, so their scores are equal if
they are summed alike, and with a budget of seven pages the lower page is in and the tail page is out.  The scores differ
from all others by more than any rounding, so the expected list is exact.  The steps go on until the cache has no room.
"""
import numpy as np
import pytest

from paper_2502_14051_amd import workloads as wl

pytestmark = pytest.mark.gpu

WINNERS, GROUP, D = 6, 4, 128
CM, TM = 0, 1  # V layouts


def run(batch, hkv, cap, tail, ps, k1, layout, slot0):
    import torch
    from paper_2502_14051_amd import rocketkv as rk
    print("[case] append tail", batch, hkv, cap, tail, ps, k1, layout, slot0, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(batch * 100003 + cap * 131 + k1 * 17 + ps)
    rnd = lambda *s: torch.randn(s, generator=gen, device=dev)
    n0 = tail * ps + slot0
    q = rnd(batch, hkv * GROUP, D).bfloat16()
    side = q.float().reshape(batch, hkv, GROUP, D).sum(2)
    side = torch.where(side < 0, -1.0, 1.0)  # the way a key has to point to score high
    twin = (side * (0.5 + torch.rand(side.shape, generator=gen, device=dev))).bfloat16()
    K = torch.empty((batch, hkv, n0, D), dtype=torch.bfloat16, device=dev).normal_(0.0, 0.05, generator=gen)
    rng = np.random.default_rng(cap + k1)
    picked = np.sort(rng.choice(tail, WINNERS + 1, replace=False))
    lower = int(picked[rng.integers(0, WINNERS + 1)])
    for p in picked:
        rows = K[:, :, p * ps:(p + 1) * ps]
        rows.copy_(twin[:, :, None] if p == lower else (4.0 * side[:, :, None] + rows.float()).bfloat16())
    K[:, :, tail * ps:] = twin[:, :, None]
    V = torch.empty_like(K).normal_(generator=gen)

    def fresh():
        c = rk.pack_cache(K, V, [n0] * batch, hkv * GROUP, ps, pages_cap=cap, v_layout=layout)
        kx, kn = rk.alloc_summaries(c)
        rk.build_page_summaries(c, kx, kn)
        if slot0 == 0:  # a page that is being opened: what its column holds is not looked at
            kx[..., tail] = 300.0
            kn[..., tail] = -300.0
        return c, kx, kn

    A, Akx, Akn = fresh()
    B, Bkx, Bkn = fresh()
    budget = (WINNERS + 1) * ps
    row = rk.pages_row_len(A, budget)
    wsA, wsB = (rk.alloc_workspace(rk.OP_HSA_DECODE, c, budget) for c in (A, B))
    outA = torch.empty((batch, hkv * GROUP, D), dtype=torch.bfloat16, device=dev)
    outB = torch.empty_like(outA)
    pgA = torch.full((batch, hkv, row), -7, dtype=torch.int32, device=dev)
    pgB = pgA.clone()
    want = torch.tensor(picked, dtype=torch.int32, device=dev).expand(batch, hkv, WINNERS + 1)
    room = min((tail + 1) * ps, cap * ps) - n0  # tokens until the tail page is full
    steps = room + (2 if tail == cap - 1 else 0)  # then two steps without room
    for s in range(steps):
        v_new = rnd(batch, hkv, D).bfloat16()
        rk.hsa_decode_append(A, q, twin, v_new, Akx, Akn, k1, budget, 0, outA, None, pgA, None, wsA)
        rk.append_kv(B, twin, v_new, Bkx, Bkn)
        rk.hsa_decode(B, q, Bkx, Bkn, k1, budget, 0, outB, None, pgB, None, wsB)
        torch.cuda.synchronize()
        assert A.seq_lens.tolist() == [n0 + min(s + 1, room)] * batch, f"step {s}"
        assert torch.equal(pgB, want), f"step {s}: the pages of the separate calls"
        assert torch.equal(pgA, want), f"step {s}: the pages of the fused step"
        assert torch.equal(outA, outB), f"step {s}: outputs"
    assert torch.equal(Akx, Bkx) and torch.equal(Akn, Bkn)
    assert torch.equal(A.k_pool, B.k_pool) and torch.equal(A.v_pool, B.v_pool)


# One, two and five pages per thread of the selection, full to the last slot, where the receiving page is also the last
# thread's own page of the last round: 512 threads, and 256 beyond 256 (sequence, KV head) units.
@pytest.mark.parametrize("batch,hkv,cap", [(4, 4, 512), (4, 4, 1024), (4, 4, 2560), (257, 1, 256), (257, 1, 512), (257, 1, 1280)])
@pytest.mark.parametrize("k1", [32, 81])
def test_last_slot(batch, hkv, cap, k1):
    run(batch, hkv, cap, cap - 1, 16, k1, CM, 0)


# three and four pages per thread, and the first cache of the next form
@pytest.mark.parametrize("batch,hkv,cap,layout", [(4, 4, 1032, CM), (4, 4, 1536, CM), (4, 4, 1544, TM), (4, 4, 2048, CM),
                                                  (4, 4, 2048, TM), (4, 4, 2056, CM), (257, 1, 520, CM), (257, 1, 768, CM),
                                                  (257, 1, 776, TM), (257, 1, 1024, CM), (257, 1, 1032, TM)])
@pytest.mark.parametrize("k1", [32, 40])
def test_three_and_four_rounds(batch, hkv, cap, layout, k1):
    run(batch, hkv, cap, cap - 1, 16, k1, layout, 0)


# the receiving page in other rounds and runs, one to 128 channels, pages already begun; token-major caches
@pytest.mark.parametrize("cap,tail,ps,k1,layout,slot0", [
    (512, 300, 16, 1, CM, 3), (512, 511, 16, 5, CM, 9), (512, 448, 16, 31, CM, 0), (512, 447, 16, 33, CM, 1),
    (520, 511, 16, 48, CM, 0), (1024, 512, 16, 128, CM, 0), (2560, 1024, 16, 40, CM, 5),
    (512, 511, 16, 32, TM, 0), (1024, 700, 7, 40, TM, 0)])
def test_places_and_channels(cap, tail, ps, k1, layout, slot0):
    run(4, 4, cap, tail, ps, k1, layout, slot0)


# more sequences than have a cache line of the workspace header each: their counters lie closer together
@pytest.mark.parametrize("batch,hkv,layout", [(128, 1, CM), (129, 1, CM), (131, 3, CM), (500, 2, CM), (131, 1, TM)])
def test_many_sequences(batch, hkv, layout):
    run(batch, hkv, 40, 39, 16, 32, layout, 0)


# six to eight pages per thread, full and not, and the first cache whose scores go through LDS
@pytest.mark.parametrize("batch,hkv,cap,tail", [(4, 4, 2568, 2567), (4, 4, 2568, 300), (4, 4, 4088, 4087), (4, 4, 4104, 4103),
                                                (257, 1, 1288, 1287), (257, 1, 2056, 2055)])
@pytest.mark.parametrize("k1", [32, 81])
def test_more_pages(batch, hkv, cap, tail, k1):
    run(batch, hkv, cap, tail, 16, k1, CM, 0)


# more pages than the register selection holds: scores through LDS.  Sequences with eight-page runs for some of the threads
# (the threads then share the rows of a run), for all but one of them, for each of them, and more than one each
@pytest.mark.parametrize("batch,hkv,cap,tail,k1,layout", [
    (4, 4, 4104, 300, 32, CM), (4, 4, 4104, 300, 81, CM), (4, 4, 4104, 2567, 81, CM), (4, 4, 4104, 4087, 32, CM),
    (4, 4, 4104, 4088, 81, CM), (4, 4, 4104, 4095, 32, CM), (1, 2, 8192, 8191, 32, CM), (1, 2, 8192, 20, 128, CM),
    (257, 1, 2056, 300, 32, CM), (257, 1, 2056, 300, 81, CM), (257, 1, 2056, 2039, 81, CM), (257, 1, 2056, 2040, 32, CM),
    (4, 4, 4104, 300, 15, TM), (257, 1, 2056, 300, 31, TM)])
def test_scores_through_lds(batch, hkv, cap, tail, k1, layout):
    run(batch, hkv, cap, tail, 16, k1, layout, 0)


# large summaries, scored by several workgroups: the receiving page in the last slot, and at either side of a share's edge
@pytest.mark.parametrize("cap,tail,ps,k1", [(3232, 3231, 3, 81), (3232, 1616, 3, 81), (3232, 1615, 3, 81), (808, 807, 3, 128),
                                            (4200, 4199, 2, 19), (8200, 8199, 1, 8), (8200, 20, 1, 9)])
def test_score_launch(cap, tail, ps, k1):
    run(4, 4, cap, tail, ps, k1, TM, 0)


# either side of the lines between one launch and several (csrc/tok_route.h): rounds of pages x (batches of 32 channels + 1)
# 12 up to 128 (sequence, KV head) units, 32 beyond; past the register selection 128 KiB of picked rows, 320 with more than
# 256 units
@pytest.mark.parametrize("batch,hkv,cap,k1", [(4, 4, 1536, 96), (4, 4, 1536, 97), (4, 4, 2560, 33), (17, 4, 1536, 128),
                                              (17, 4, 2560, 64), (17, 4, 2560, 65), (33, 4, 4096, 96), (33, 4, 4096, 97),
                                              (257, 1, 2048, 96), (257, 1, 2048, 97), (4, 4, 4104, 15), (4, 4, 4104, 16),
                                              (257, 1, 2064, 79), (257, 1, 2064, 80),
                                              (4, 4, 2048, 64), (4, 4, 2048, 65), (32, 4, 3072, 32), (32, 4, 3584, 32)])
def test_one_launch_or_several(batch, hkv, cap, k1):
    run(batch, hkv, cap, cap - 1, 2, k1, TM, 0)


# six, seven and eight rounds, full and not
@pytest.mark.parametrize("cap,tail", [(3072, 3071), (3080, 3079), (3584, 3583), (3592, 1500), (4096, 4095)])
def test_six_to_eight_rounds(cap, tail):
    run(4, 4, cap, tail, 16, 32, CM, 0)
