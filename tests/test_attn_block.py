"""GPU tests of the drafter attention's one-kernel route for short key ranges
(needs an MI355X), against the float64 oracle within the tolerance derived in
test_attn: the edges of its 32-key units and of the rule that chooses it.
"""

import pytest

from paper_2607_04244_amd import qlin
from test_attn import case, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (32, 8), (6, 2), (21, 3), (64, 8)])
@pytest.mark.parametrize("nq,T,W", [(1, 1, 0), (16, 31, 0), (7, 32, 0), (16, 33, 0), (16, 64, 0), (5, 97, 0),
                                    (16, 300, 20), (16, 1000, 512), (3, 319, 0), (16, 320, 0), (16, 700, 101)])
def test_short_ranges_run_in_one_kernel(Hq, Hkv, nq, T, W):
    S, ws, text = qlin.qlin_swa_plan(Hq, Hkv, 128, nq, T, W)
    assert "kernel=k_attn_block" in text and "combine=0" in text and (S, ws) == (1, 0), text
    q, k, v = case(Hq, Hkv, nq, T, kv_stride=T + 5, seed=Hq + T + W)
    k[:, T:] = 0x7FC0                      # beyond T: NaN, never read
    v[:, T:] = 0x7FC0
    check(q, k, v, T, W, what=f"{Hq}/{Hkv} nq={nq} T={T} W={W}")


@pytest.mark.parametrize("Hq,Hkv,T,block", [(32, 8, 321, False), (64, 8, 321, True), (64, 8, 384, True),
                                            (64, 8, 385, False), (65, 13, 64, False), (72, 9, 300, False)])
def test_rule_edges(Hq, Hkv, T, block):
    text = qlin.qlin_swa_plan(Hq, Hkv, 128, 16, T, 0)[2]
    assert ("k_attn_block" in text) == block, text
    q, k, v = case(Hq, Hkv, 16, T, seed=T)
    check(q, k, v, T, 0, what=f"{Hq}/{Hkv} T={T}")


def test_forced_single_split_keeps_its_kernel():
    assert "k_attn_split<1,4>" in qlin.qlin_swa_plan(32, 8, 128, 16, 100, 0, 1)[2]
