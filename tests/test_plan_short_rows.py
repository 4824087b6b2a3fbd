"""Decode rows of a few blocks in the host plan (CPU): they are read whole, with
no partial results and no merge, where the launch fits one generation of waves
as it is or the steps that a cut would save are fewer than a merge costs."""
import ctypes

import numpy as np
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


def _rule(lens, wpd, light):
    """Longest piece of unshared rows of `lens` blocks in one generation of waves
    (12 per CU x 256 CUs), by trying every length; None past one generation."""
    step = ((28, 43, 62), (28, 30, 44))[light]
    default = 96 if light else 48
    units = sum(lens) * wpd // 2048
    target = max(8, min(default, units))
    longest = max(target, min(4 * default, units))
    waves = lambda sp: sum(-(-n // sp) for n in lens) * wpd  # noqa: E731
    if waves(longest) > 3072:
        return None
    best, split = 1 << 62, target
    for per_cu in (1, 2, 3):
        fit = [sp for sp in range(6, max(longest, default) + 1) if waves(sp) <= 1024 * per_cu]
        if fit and 10 * step[per_cu - 1] * ((fit[0] + 1) // 2) < 9 * best:
            best, split = step[per_cu - 1] * ((fit[0] + 1) // 2), fit[0]
    whole = max(lens)
    if whole > split and step[-(-waves(whole) // 1024) - 1] * ((whole + 1) // 2) <= best + 80:
        split = whole
    return max(-(-n // -(-n // split)) for n in lens)


@pytest.mark.parametrize("hq,hkv,d,kv", [(32, 8, 128, W.KV_BF16), (4, 4, 128, W.KV_BF16),
                                         (32, 32, 128, W.KV_BF16), (32, 8, 128, W.KV_FP8)])
def test_pieces_are_the_shortest_that_fit(hq, hkv, d, kv):
    rng, checked = np.random.default_rng(5), 0
    for n in (1, 2, 3, 5, 8, 17, 40, 64, 100, 250):
        for top in (3, 9, 20, 60, 200):
            lens = rng.integers(1, top + 1, n).tolist()
            want = _rule(lens, hkv, kv != W.KV_BF16)
            if want is None:
                continue
            w = W.build("rule", [W.RowSpec(W.DECODE, 16 * k - 1, 1) for k in lens], {}, hq, hkv, d,
                        kv_dtype=kv, seed=3, values=False)
            cp, cb, _keep = echo.host_structs(w)
            lay, words = echo.plan_pack(cp, cb, hq)
            p = words[lay["off_desc"]:lay["off_desc"] + 8 * lay["n_desc"]].reshape(-1, 8)
            assert ((p[:, 4] - p[:, 3] + 15) // 16).max() == want, (n, top)
            checked += 1
    assert checked > 25
