"""The merge's two forms, a wave per head and a wave for four, at the edges of
their rules, against the fp64 oracle: rows of 15 to 17, 63 to 65 and 129 entries
(a 16-lane group's turn, a wave's turn), few and many (token, head) pairs, head
counts that four does not divide."""
import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import ATOL, attn_error, say

pytestmark = pytest.mark.gpu

# decode rows whose contexts are cut into many pieces beside short ones
LONG = [W.RowSpec(W.DECODE, c, 1) for c in (2000, 2060, 2200, 8000, 8200, 8400, 17000)]
SHORT = [W.RowSpec(W.DECODE, 150 + 7 * i, 1) for i in range(90)]


@pytest.mark.parametrize("mirrors", [True, False])
@pytest.mark.parametrize("d,kv", [(64, W.KV_BF16), (128, W.KV_BF16), (128, W.KV_FP8)])
@pytest.mark.parametrize("rows,hq,hkv", [("long", 6, 2), ("both", 30, 2), ("one", 3, 3)])
def test_merge_forms(rows, hq, hkv, d, kv, mirrors):
    import torch
    from paper_2504_03651_amd.session import Iteration
    r = {"long": LONG, "both": LONG + SHORT, "one": LONG[-1:]}[rows]
    w = W.build(f"merge-{rows}", r, {}, hq, hkv, d, kv_dtype=kv, seed=97)
    say(f"[case] merge {rows} {hq}/{hkv} D={d} {kv} mirrors={mirrors}")
    it = Iteration(w, mirrors=mirrors)
    it.out.fill_(float("nan"))
    it.step()
    torch.cuda.synchronize()
    _, ref = oracle.run_iteration(w)
    err, _ = attn_error(it.out.cpu().numpy().reshape(ref.shape), ref)
    say(f"       max abs err {err:.3e}")
    assert err <= ATOL
