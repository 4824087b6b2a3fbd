"""Chunked prefill at head_dim 64 on both sides of the rule that puts two
workgroups on a CU (more than 512 workgroups on 256 CUs), against the fp64
oracle: ragged chunks whose tiles end inside and on the 64-key tiles, with
logits of ordinary size and 16 times that (the softmax reference moves)."""
import numpy as np
import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import ATOL, attn_error, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv", [W.KV_BF16, W.KV_FP8])
@pytest.mark.parametrize("hq,hkv,rows", [(16, 16, 32), (16, 16, 33), (64, 8, 70), (24, 8, 65)])
@pytest.mark.parametrize("factor", [1.0, 16.0])
def test_prefill_dense_rule(hq, hkv, rows, kv, factor):
    import torch
    from paper_2504_03651_amd.session import Iteration
    # one tile per row: rows x hkv workgroups
    n = 256 // (hq // hkv)
    r = [W.RowSpec(W.PREFILL, (0, 63, 64, 200, 447)[i % 5], 2 + (37 * i) % (n - 1)) for i in range(rows)]
    w = W.build(f"dense-{rows}x{hkv}", r, {}, hq, hkv, 64, kv_dtype=kv, seed=83)
    x = (w.q.astype(np.uint32) << 16).view(np.float32) * np.float32(factor)   # exact in bf16
    w.q = (x.view(np.uint32) >> 16).astype(np.uint16)
    for mirrors in (True, False):
        say(f"[case] dense prefill {rows} x {hkv} heads {kv} x{factor:g} mirrors={mirrors}")
        it = Iteration(w, mirrors=mirrors)
        it.step()
        torch.cuda.synchronize()
        if mirrors:
            _, ref = oracle.run_iteration(w)
        err, _ = attn_error(it.out.cpu().numpy().reshape(ref.shape), ref)
        say(f"       max abs err {err:.3e}")
        assert err <= ATOL
