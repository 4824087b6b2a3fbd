"""Decode rows of a few blocks in the host plan (CPU): they are read whole, with
no partial results and no merge, where the launch fits one generation of waves
as it is or the steps that a cut would save are fewer than a merge costs."""
import ctypes

import pytest

from paper_2504_03651_amd import echo
from paper_2504_03651_amd import workload as W

LAYOUTS = [(32, 8, 128, W.KV_BF16), (16, 16, 128, W.KV_BF16), (32, 32, 128, W.KV_BF16),
           (64, 8, 64, W.KV_BF16), (32, 8, 128, W.KV_FP8)]


def _stats(rows, hq, hkv, d, kv):
    w = W.build("short", rows, {}, hq, hkv, d, kv_dtype=kv, seed=3, values=False)
    cp, cb, _keep = echo.host_structs(w)
    st = echo.CPlanStats()
    assert echo.lib().echo_attn_plan_stats(ctypes.byref(cp), ctypes.byref(cb), hq,
                                           ctypes.byref(st)) == echo.ECHO_OK
    return st


@pytest.mark.parametrize("hq,hkv,d,kv", LAYOUTS)
def test_rows_of_a_few_blocks_stay_whole(hq, hkv, d, kv):
    for blocks in range(1, 11):
        for n in (1, 2, 8, 16, 33, 56, 64, 96, 110, 128, 150, 193, 200, 240, 255, 300):
            rows = [W.RowSpec(W.DECODE, 16 * blocks - 1 - i % 8, 1) for i in range(n)]
            st = _stats(rows, hq, hkv, d, kv)
            if n * hkv <= 3072:
                assert st.partial_slots == 0 and st.decode_items == n * hkv, (blocks, n)


def test_rows_past_one_generation_are_cut_no_shorter_than_eight_blocks():
    # 400 rows x 8 heads are past 3,072 waves, with few blocks in all
    rows = [W.RowSpec(W.DECODE, 127 if i % 4 == 0 else 31, 1) for i in range(400)]
    assert _stats(rows, 32, 8, 128, W.KV_BF16).partial_slots == 0


def test_long_rows_are_cut_all_the_same():
    for hq, hkv, d, kv in LAYOUTS:
        st = _stats([W.RowSpec(W.DECODE, 16 * 24 - 1, 1)] * 8, hq, hkv, d, kv)
        assert st.partial_slots > 0
    # a chunk whose keys are cut needs the merge in any case
    chunk = [W.RowSpec(W.PREFILL, 3000, 40)]
    st = _stats([W.RowSpec(W.DECODE, 127, 1)] * 8 + chunk, 32, 8, 128, W.KV_BF16)
    assert st.decode_items == 2 * 8 * 8
