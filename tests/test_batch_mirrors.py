"""Host state that calls keep or check (CPU): the addresses a DeviceBatch passes
for its host mirrors follow the arrays, also after a mirror was replaced and in a
copy of the batch; the block copy's check of its pairs; the ring of host buffers;
the size of a device-built plan against the static entry point's scratch."""
import copy
import ctypes

import numpy as np
import pytest
import torch

from paper_2504_03651_amd import echo
from paper_2504_03651_amd import workload as W


def _addresses(b):
    c = b.c()
    return c.h_block_tables, c.h_seq_lens, c.h_q_start, c.h_row_kind


def _want(b):
    return tuple(a.ctypes.data for a in (b.h_bt, b.h_sl, b.h_qs, b.h_kind))


def test_mirror_addresses_follow_the_arrays():
    b = echo.DeviceBatch(W.config1().batch, "cpu")
    assert _addresses(b) == _want(b) == _addresses(b)
    b.h_sl = b.h_sl + 0
    assert _addresses(b) == _want(b)
    for twin in (copy.copy(b), copy.deepcopy(b)):
        assert _addresses(twin) == _want(twin)
    b.mirrors = False
    assert _addresses(b) == (None,) * 4


@pytest.mark.parametrize("blocks", [64, (1 << 20) + 1, 2 ** 31 - 1])
def test_block_copy_pairs_are_checked_in_any_order(blocks):
    # one pass over the pairs finds what sorting found: a destination twice, a
    # block on both sides in either order; pools of many blocks are sorted
    pool = echo.CPool(0x1000, 0x1000, None, None, blocks, 2, 64, 16, echo.KV_BF16)

    def call(pairs):
        h = np.ascontiguousarray(pairs, np.int32)
        return echo.lib().echo_block_copy(ctypes.byref(pool), 0x1000, len(h), h.ctypes.data, None)

    for bad in ([(1, 5), (2, 5)], [(1, 5), (5, 6)], [(5, 6), (1, 5)], [(3, 3)],
                [(1, 5), (2, 6), (7, 1)], [(1, 5), (2, 6), (6, 8), (9, 5)]):
        assert call(bad) == echo.ECHO_E_INVALID, bad
    assert call([(-1, 3)]) == echo.ECHO_E_RANGE
    if blocks < 2 ** 31 - 1:
        assert call([(1, blocks)]) == echo.ECHO_E_RANGE


def test_each_buffer_of_the_ring_grows_once(monkeypatch):
    # a plan larger than a new buffer: the first use of each buffer is refused
    # and grows it, and from then on every call plans once
    need, calls, kept = 100_000, [], []

    class Lib:
        def hipHostMalloc(self, p, size, flags):
            kept.append(ctypes.create_string_buffer(size.value))
            ctypes.cast(p, ctypes.POINTER(ctypes.c_void_p))[0] = ctypes.addressof(kept[-1])
            return 0

        def hipHostFree(self, p):
            return 0

        def echo_attn_host_workspace_bytes(self, *a):
            return need

        def echo_attn_mixed(self, *a):
            calls.append(a[8])
            return echo.ECHO_OK if a[9] >= need else echo.ECHO_E_WORKSPACE

        def echo_last_error(self):
            return b""

    class Stream:
        cuda_stream = 0

    fake = Lib()
    monkeypatch.setattr(echo, "lib", lambda: fake)
    w = W.config1()
    pool = echo.KVPool(w.num_blocks, w.num_kv_heads, w.head_dim, False, "cpu")
    b = echo.DeviceBatch(w.batch, "cpu")
    t = torch.zeros(4)
    hw = echo.HostWorkspace()
    monkeypatch.setattr(hw, "release", lambda slot, stream: None)
    for i in range(12):
        before = len(calls)
        echo.attn_mixed(pool, b, t, w.num_q_heads, 1.0, t, t, Stream(), hw)
        assert len(calls) - before == (2 if i < 4 else 1), i


def test_device_plan_regions_fit_the_static_scratch():
    # 2,040 rows of at most 7 blocks and 16 heads: regions for pieces of 6 blocks
    # (two a row) would outgrow the static entry point's 32 MiB
    pool = echo.CPool(0x1000, 0x1000, None, None, 20000, 1, 128, 16, echo.KV_BF16)
    b = echo.CBatch(2040, 7, 2040, 1, 112, 0x1000, 0x1000, 0x1000, 0x1000)
    n = echo.lib().echo_attn_workspace_bytes(ctypes.byref(pool), ctypes.byref(b), 16)
    assert 0 < n <= 32 << 20
