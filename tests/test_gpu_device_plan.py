"""The device-built plan at the edges of its windows and launch forms, against
the fp64 oracle: rows and block ids at the limits of the one-workgroup form
(1,024 rows, 32,768 ids) and one past them, a descriptor region of one piece
per row, and prefill rows of one token, which are decode work."""
import numpy as np
import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import ATOL, attn_error, say

pytestmark = pytest.mark.gpu


def _short(n):
    return [W.RowSpec(W.DECODE, (7 * i) % 45, 1) if i % 5 else W.RowSpec(W.PREFILL, (3 * i) % 20, 1 + i % 4)
            for i in range(n)]


def _long(n):
    # one row of 2,048 blocks sets the width of every row's table
    return [W.RowSpec(W.DECODE, 32767, 1)] + [W.RowSpec(W.DECODE, 40 + 100 * i, 1) for i in range(n - 1)]


CASES = {
    "one-row": [W.RowSpec(W.DECODE, 0, 1)],
    "rows-1024": _short(1024),
    "rows-1025": _short(1025),
    "ids-32768": _long(16),
    "ids-34816": _long(17),
    "one-piece-per-row": [W.RowSpec(W.DECODE, c, 1) for c in (0, 15, 16, 100, 127)],
    "one-token-chunks": [W.RowSpec(W.PREFILL, c, 1) for c in (0, 15, 16, 700)] +
                        [W.RowSpec(W.DECODE, 300, 1)],
    "one-token-beside-chunks": [W.RowSpec(W.PREFILL, 500, 1), W.RowSpec(W.PREFILL, 70, 130),
                                W.RowSpec(W.DECODE, 900, 1), W.RowSpec(W.PREFILL, 0, 1)],
}


@pytest.mark.parametrize("kv", [W.KV_BF16, W.KV_FP8])
@pytest.mark.parametrize("name", list(CASES))
def test_device_plan_edges(name, kv):
    import torch
    from paper_2504_03651_amd.session import Iteration
    w = W.build(name, CASES[name], {}, 4, 2, 64, kv_dtype=kv, seed=61)
    say(f"[case] device plan {name} {kv}: rows={w.batch.num_rows} T={w.batch.num_tokens}")
    it = Iteration(w, mirrors=False)
    it.out.fill_(float("nan"))
    it.step()
    torch.cuda.synchronize()
    hdr = it.workspace[:64 * 4].view(torch.int32).cpu().numpy()
    assert hdr[4] == 0, "no row may be skipped"
    _, ref = oracle.run_iteration(w)
    err, _ = attn_error(it.out.cpu().numpy().reshape(ref.shape), ref)
    say(f"       max abs err {err:.3e}")
    assert err <= ATOL


def test_only_the_rows_that_get_no_work_are_counted_as_skipped():
    # max_q_len 1 leaves no room for prefill tiles: the row of four tokens is
    # skipped, and the decode rows after it are computed and not counted
    import torch
    from paper_2504_03651_amd.session import Iteration
    rows = [W.RowSpec(W.DECODE, 300, 1), W.RowSpec(W.PREFILL, 20, 4)] + \
           [W.RowSpec(W.DECODE, c, 1) for c in (500, 40, 900)]
    w = W.build("skipped", rows, {}, 4, 2, 64, seed=67)
    say("[case] device plan, a row that does not fit")
    it = Iteration(w, mirrors=False)
    it.copy()
    it.append()
    it.batch.max_q_len = 1
    it.out.fill_(7.0)
    it.attend()
    torch.cuda.synchronize()
    hdr = it.workspace[:64 * 4].view(torch.int32).cpu().numpy()
    assert hdr[4] == 1
    _, ref = oracle.run_iteration(w)
    got = it.out.cpu().numpy()
    ref = ref.reshape(got.shape)
    assert (got[1:5] == 7.0).all()
    keep = [0, 5, 6, 7]
    err, _ = attn_error(got[keep], ref[keep])
    say(f"       max abs err {err:.3e}")
    assert err <= ATOL
