"""GPU tests of the drafter attention's one-kernel route for short key ranges
and of the split whose workgroups share a key/value head's query heads (needs
an MI355X), against the float64 oracle within the tolerance derived in
test_attn: the edges of the 32-key units and of the rules.
"""

import numpy as np
import pytest
import torch

from oracle import attn_ref as ar
from paper_2607_04244_amd import qlin
from test_attn import case, check, host_f64, run, tolerance

pytestmark = pytest.mark.gpu


def planned(ok, text):
    """A statement about the plan, which compares head counts with the compute
    units of the device it was measured on."""
    assert ok or torch.cuda.get_device_properties(0).multi_processor_count != 256, text


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (32, 8), (6, 2), (21, 3), (64, 8)])
@pytest.mark.parametrize("nq,T,W", [(1, 1, 0), (16, 31, 0), (7, 32, 0), (16, 33, 0), (16, 64, 0), (5, 97, 0),
                                    (16, 300, 20), (16, 1000, 512), (3, 319, 0), (16, 320, 0), (16, 700, 101)])
def test_short_ranges_run_in_one_kernel(Hq, Hkv, nq, T, W):
    S, ws, text = qlin.qlin_swa_plan(Hq, Hkv, 128, nq, T, W)
    planned("kernel=k_attn_block" in text and "combine=0" in text and (S, ws) == (1, 0), text)
    q, k, v = case(Hq, Hkv, nq, T, kv_stride=T + 5, seed=Hq + T + W)
    k[:, T:] = 0x7FC0                      # beyond T: NaN, never read
    v[:, T:] = 0x7FC0
    check(q, k, v, T, W, what=f"{Hq}/{Hkv} nq={nq} T={T} W={W}")


@pytest.mark.parametrize("Hq,Hkv,T,block", [(32, 8, 321, False), (64, 8, 321, True), (64, 8, 384, True),
                                            (64, 8, 385, False), (65, 13, 64, False), (72, 9, 300, False)])
def test_rule_edges(Hq, Hkv, T, block):
    text = qlin.qlin_swa_plan(Hq, Hkv, 128, 16, T, 0)[2]
    planned(("k_attn_block" in text) == block, text)
    q, k, v = case(Hq, Hkv, 16, T, seed=T)
    check(q, k, v, T, 0, what=f"{Hq}/{Hkv} T={T}")


@pytest.mark.parametrize("Hq,Hkv,nq,T,W", [(5, 1, 16, 700, 0), (12, 2, 9, 2000, 1024), (21, 3, 16, 1000, 0),
                                           (64, 8, 16, 1300, 0), (128, 16, 16, 500, 0), (40, 8, 1, 385, 0)])
def test_two_workgroups_share_a_heads_queries(Hq, Hkv, nq, T, W):
    S, ws, text = qlin.qlin_swa_plan(Hq, Hkv, 128, nq, T, W)
    planned("k_attn_split<1,4>" in text and f"grid={2 * Hkv * S} " in text, text)
    q, k, v = case(Hq, Hkv, nq, T, seed=Hq + T)
    check(q, k, v, T, W, what=f"{Hq}/{Hkv} nq={nq} T={T} W={W}")


def test_too_many_heads_to_share_keep_two_heads_a_wave():
    text = qlin.qlin_swa_plan(160 * 5, 160, 128, 16, 400, 0)[2]
    planned("k_attn_split<2,3>" in text, text)
    q, k, v = case(160 * 5, 160, 4, 400, seed=3)
    check(q, k, v, 400, 0, what="160 key/value heads")


def test_forced_single_split_keeps_its_kernel():
    assert "k_attn_split<1,4>" in qlin.qlin_swa_plan(32, 8, 128, 16, 100, 0, 1)[2]


@pytest.mark.parametrize("Hq,Hkv,T,kernel,splits", [
    (520, 65, 2064, "<2,3>", 3),       # one range for three would be half as long again
    (360, 72, 8192, "<2,3>", 3),
    (120, 24, 8192, "<2,3>", 10),      # long ranges
    (320, 64, 8192, "<2,3>", 4),
    (520, 65, 700, "<1,4>", 1),        # short: one range, no combination
    (768, 96, 2064, "<1,4>", 1), (768, 96, 5000, "<2,3>", 2), (800, 100, 2064, "<2,3>", 2),
    (64, 8, 8192, "<1,4>", 16), (8, 1, 16000, "<1,4>", 125),
])
def test_when_two_workgroups_share_a_head(Hq, Hkv, T, kernel, splits):
    """The measured choice between two workgroups a (head, range) and two heads
    a wave, and that the chosen plan covers every key."""
    S, ws, text = qlin.qlin_swa_plan(Hq, Hkv, 128, 16, T, 0)
    planned("k_attn_split" + kernel in text and S == splits, text)
    if Hq * T < 10 ** 6:
        q, k, v = case(Hq, Hkv, 2, T, seed=T)
        check(q, k, v, T, 0, what=f"{Hq}/{Hkv} T={T}")


@pytest.mark.parametrize("T", [100, 300, 700])
def test_infinite_keys_and_values(T):
    """A key of -infinity under positive queries has weight zero, and an
    infinite value stays in its dimension (infinite, or NaN where its weight is
    zero in bf16), in one kernel and in the split."""
    Hq, Hkv, nq = 8, 2, 16
    q, k, v = case(Hq, Hkv, nq, T, seed=T)
    q = np.maximum(q & 0x7FFF, 0x3C00).astype(np.uint16)            # positive
    k[:, 7] = 0xC640                                                # -12288: the weight vanishes as well
    ref = ar.swa_attention(q, k[:, :T], v[:, :T], 0)
    k[:, 7] = 0                                                     # a key without weight adds no error
    tol = tolerance(q, k, v, T, 0, ref)
    k[:, 7] = 0xFF80
    v[:, 50, 3] = 0x7F80
    got = host_f64(run(q, k, v, T, 0))
    rest = np.arange(128) != 3
    assert np.all(np.abs(got - ref)[..., rest] <= tol[..., rest])
    assert not np.isfinite(got[..., 3]).any() and not np.isneginf(got[..., 3]).any()
