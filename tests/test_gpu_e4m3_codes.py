"""The append's e4m3 codes for every bf16 value (infinities, NaN, zeros of both
signs, subnormals and all rounding ties among them), bit for bit against the
oracle's encoder, at scales that the rounded quotient is taken by its reciprocal
for and at ones that it is divided for: blocks written in part and single slots,
whose scales stand in the pool."""
import numpy as np
import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import same_pool, say

pytestmark = pytest.mark.gpu

# per KV head; 2^-120 and 2^110 lie outside the range of the reciprocal, 0.75 puts
# the quotients of bf16 values between the codes, 2^-1 and 1 on their ties
SCALES = np.array([1.0, 0.5, 0.75, 3.0 / 448, 2.0 ** -100, 2.0 ** 100, 2.0 ** -120, 2.0 ** 110], np.float32)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("slots", [15, 7, 1])
def test_every_bf16_value(d, slots):
    import torch
    from paper_2504_03651_amd.session import Iteration
    H = len(SCALES)
    n = -(-65536 // (slots * d))                       # rows that hold every value once
    # slot 0 is cached, so the block keeps its scale
    rows = [W.RowSpec(W.PREFILL, 1 + (i % (16 - slots)), slots) for i in range(n)]
    w = W.build(f"codes-{slots}", rows, {}, H, H, d, kv_dtype=W.KV_FP8, seed=73)
    say(f"[case] e4m3 codes D={d} slots={slots}: rows={n}")
    # [T][H][D]: head h takes the values in its own order; V against K reversed
    x = (np.arange(n * slots * d) % 65536).astype(np.uint16).reshape(-1, 1, d)
    x = np.concatenate([(x + np.uint16(h * 257)) for h in range(H)], 1)
    w.k_new, w.v_new = np.ascontiguousarray(x), np.ascontiguousarray(x[::-1])
    pool = oracle.prepare(w)
    it = Iteration(w)
    for s, t, p in ((SCALES, it.pool.k_scale, pool.k_scale), (SCALES[::-1], it.pool.v_scale, pool.v_scale)):
        p[:] = s
        t.copy_(torch.from_numpy(np.ascontiguousarray(p)))
    oracle.kv_append(pool, w.batch, w.k_new, w.v_new)
    it.append()
    torch.cuda.synchronize()
    same_pool(it.pool_host(), pool)
