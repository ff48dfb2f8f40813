"""Lists whose wavefronts walk more than one pair.  Shared equally (list_shares): 33, 44, 48 and 49 entries over two
workgroups of eight wavefronts, a list shorter than its row.  In whole rounds of the wavefronts, with more
workgroups than run at once: 44 and 75 entries over eight wavefronts, 37 and 65 over four.  Both V
layouts, against the oracle (attention 1e-2, selections within a 1e-3 band)."""
import pytest

from paper_2502_14051_amd import workloads as wl
from test_gpu_token_major import TM, decode_and_check, env, say, small  # noqa: F401 (env: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, TM])
@pytest.mark.parametrize("units,budget,lens", [
    (104, 33 * 16, None), (104, 44 * 16, None), (104, 777, (1200, 300, 17)), (100, 49 * 16, None),
    (160, 44 * 16, None), (132, 75 * 16, (1200, 1100)), (260, 37 * 16, None), (260, 65 * 16, (1200, 1100)),
])
def test_shares(env, oracle, layout, units, budget, lens):
    hkv = 4
    w = small("tiny", batch=units // hkv, n_q_heads=8, n_kv_heads=hkv, context=1200, token_budget=budget, n_heavy=4)
    say("list shares", layout, units, budget, lens)
    d = wl.generate(w)
    if lens is not None:
        d["seq_lens"][:len(lens)] = lens
    decode_and_check(env, oracle, w, d, 0, 7, v_layout=layout)
