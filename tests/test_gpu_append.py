"""The append's two launch forms at their edges, bit for bit against the
oracle: every first slot and token count of a block written in part, and row
counts around the 64-way search for a unit's row (64 and 4,096 rows)."""
import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import same_pool, say

pytestmark = pytest.mark.gpu

# slot s of the first block and q tokens: one block in part, whole, two, three
EDGES = [W.RowSpec(W.PREFILL, 16 * (s % 3) + s, q) for s in range(16) for q in (1, 2, 15, 16, 17, 33)]


def _check(name, rows, hq, hkv, d, kv):
    import torch
    from paper_2504_03651_amd.session import Iteration
    w = W.build(name, rows, {}, hq, hkv, d, kv_dtype=kv, seed=71)
    say(f"[case] append {name} {hkv}x{d} {kv}: rows={w.batch.num_rows} T={w.batch.num_tokens}")
    it = Iteration(w)
    it.append()
    torch.cuda.synchronize()
    pool = oracle.prepare(w)
    oracle.kv_append(pool, w.batch, w.k_new, w.v_new)
    same_pool(it.pool_host(), pool)


@pytest.mark.parametrize("kv", [W.KV_BF16, W.KV_FP8])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("long", [False, True])
def test_append_block_edges(d, kv, long):
    # one long chunk pads the direct form past its bound: units by number then
    _check("long" if long else "short", EDGES + ([W.RowSpec(W.PREFILL, 5, 3000)] if long else []),
           3, 3, d, kv)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4096, 4097])
def test_append_row_search(n):
    rows = [W.RowSpec(W.PREFILL, (5 * i) % 37, 1 + (i % 7) * (i % 5)) for i in range(n - 1)]
    _check(f"rows-{n}", rows + [W.RowSpec(W.PREFILL, 9, 16 * n + 700)], 2, 1, 64, W.KV_BF16)


@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1])
def test_append_grid_limit(n):
    # rows x 32 heads on both sides of 2^26 units, where the direct form's grid
    # would reach 2^32 threads.  Four rows hold blocks; the others name block -1,
    # which the kernels skip without reading their tokens.
    import ctypes

    import torch
    from paper_2504_03651_amd import echo
    say(f"[case] append {n} rows x 32 heads")
    pool = echo.KVPool(8, 32, 64).poison()
    at = [0, 77, n // 2, n - 1]
    bt = torch.full((n, 1), -1, dtype=torch.int32, device="cuda")
    for i, r in enumerate(at):
        bt[r, 0] = 2 * i
    sl = torch.ones(n, dtype=torch.int32, device="cuda")
    qs = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    kind = torch.zeros(n, dtype=torch.uint8, device="cuda")
    k = torch.empty(n, 32, 64, dtype=torch.int16, device="cuda")
    v = torch.empty_like(k)
    for t in (k, v):
        t[at] = torch.randint(0, 1 << 14, (4, 32, 64), device="cuda").short()
    cp = pool.c()
    cb = echo.CBatch(n, 1, n, 1, 1, bt.data_ptr(), sl.data_ptr(), qs.data_ptr(), kind.data_ptr())
    rc = echo.lib().echo_kv_append(ctypes.byref(cp), ctypes.byref(cb), k.data_ptr(), v.data_ptr(),
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == echo.ECHO_OK, echo.last_error()
    torch.cuda.synchronize()
    for i, r in enumerate(at):
        assert torch.equal(pool.k[2 * i, :, 0], k[r]) and torch.equal(pool.v[2 * i, :, :, 0], v[r])
    assert (pool.k[:, :, 1:] == 0x7FC0).all() and (pool.k[1::2] == 0x7FC0).all()
    assert (pool.v[..., 1:] == 0x7FC0).all() and (pool.v[1::2] == 0x7FC0).all()
