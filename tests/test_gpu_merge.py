"""The merge's two forms, a wave per head and a wave for four, at the edges of
their rules, against the fp64 oracle: rows of 15 to 17, 63 to 65, 128 and 129
entries (a 16-lane group's turn, a wave's turn; past 16 a head gets a wave), few
and many (token, head) pairs, head counts that four does not divide.  The entries
are counted in the plan, so that another piece length shows up here."""
import pytest

import oracle
from paper_2504_03651_amd import echo
from paper_2504_03651_amd import workload as W
from tests.gpu_util import ATOL, attn_error, say

PIECE = 6      # blocks per decode piece of these batches
COUNTS = (15, 16, 17, 63, 64, 65, 128, 129)
# decode rows of that many pieces (the last one a few keys short) beside short ones
LONG = [W.RowSpec(W.DECODE, 16 * PIECE * n - 1 - n % 11, 1) for n in COUNTS]
SHORT = [W.RowSpec(W.DECODE, 150 + 7 * i, 1) for i in range(90)]
ROWS = {"long": LONG, "both": LONG + SHORT, "one": LONG[-1:]}
SHAPES = [("long", 6, 2), ("both", 30, 2), ("one", 3, 3)]
KINDS = [(64, W.KV_BF16), (128, W.KV_BF16), (128, W.KV_FP8)]


def _pieces(rows):
    return [-(-(r.ctx + 1) // (16 * PIECE)) for r in rows]


def _build(rows, hq, hkv, d, kv, values=True):
    return W.build(f"merge-{rows}", ROWS[rows], {}, hq, hkv, d, kv_dtype=kv, seed=97, values=values)


@pytest.mark.parametrize("d,kv", KINDS)
@pytest.mark.parametrize("rows,hq,hkv", SHAPES)
def test_entries_per_row(rows, hq, hkv, d, kv):
    w = _build(rows, hq, hkv, d, kv, values=False)
    cp, cb, _keep = echo.host_structs(w)
    lay, words = echo.plan_pack(cp, cb, hq)
    n = lay["n_merge_rows"]
    tok = words[lay["off_merge_tok"]:lay["off_merge_tok"] + n]
    ptr = words[lay["off_merge_ptr"]:lay["off_merge_ptr"] + n + 1]
    got = {int(t): int(b - a) for t, a, b in zip(tok, ptr, ptr[1:])}
    want = {t: p for t, p in enumerate(_pieces(ROWS[rows])) if p > 1}
    assert got == want


@pytest.mark.gpu
@pytest.mark.parametrize("mirrors", [True, False])
@pytest.mark.parametrize("d,kv", KINDS)
@pytest.mark.parametrize("rows,hq,hkv", SHAPES)
def test_merge_forms(rows, hq, hkv, d, kv, mirrors):
    import torch
    from paper_2504_03651_amd.session import Iteration
    w = _build(rows, hq, hkv, d, kv)
    say(f"[case] merge {rows} {hq}/{hkv} D={d} {kv} mirrors={mirrors}")
    it = Iteration(w, mirrors=mirrors)
    it.out.fill_(float("nan"))
    it.step()
    torch.cuda.synchronize()
    if not mirrors:   # the header's merged rows and partial slots (one per entry and head)
        hdr = it.workspace[:64 * 4].view(torch.int32).cpu().numpy()
        want = [p for p in _pieces(ROWS[rows]) if p > 1]
        assert hdr[2] == len(want)
        # (one row alone: its region holds pieces of 8 blocks)
        assert hdr[3] == (97 if rows == "one" else sum(want)) * hq
    _, ref = oracle.run_iteration(w)
    err, _ = attn_error(it.out.cpu().numpy().reshape(ref.shape), ref)
    say(f"       max abs err {err:.3e}")
    assert err <= ATOL
