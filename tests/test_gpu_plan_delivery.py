"""How a host-built plan reaches the kernels: the decode kernel of a launch of
one generation of waves reads it in pinned host memory and copies it for the
kernels after it; larger launches, and those beside a large prefill, copy it
first.  Both sides of that rule (3,072 waves, 512 prefill workgroups on 256
CUs), with and without chunks and merges, against the oracle; batches of different
plans through one buffer and through the ring, with nothing waited for in between;
and a captured call replayed with other work in between, against the eager
result."""
import ctypes

import pytest

import oracle
from paper_2504_03651_amd import workload as W
from tests.gpu_util import ATOL, attn_error, say

pytestmark = pytest.mark.gpu

CHUNK = [W.RowSpec(W.PREFILL, 100, 70)]
CASES = {
    # 32 KV heads: 96 rows of one piece are 3,072 waves
    "direct": [W.RowSpec(W.DECODE, 20 + i % 60, 1) for i in range(96)],
    "copied": [W.RowSpec(W.DECODE, 20 + i % 60, 1) for i in range(97)],
    "direct-chunk": [W.RowSpec(W.DECODE, 20 + i, 1) for i in range(40)] + CHUNK,
    "copied-chunk": [W.RowSpec(W.DECODE, 20 + i, 1) for i in range(97)] + CHUNK,
    "direct-merge": [W.RowSpec(W.DECODE, 900 + 90 * i, 1) for i in range(4)] + CHUNK,
    "chunk-only": CHUNK,
    # a chunk is one tile: 512 prefill workgroups (two rounds of CUs), and 544
    "direct-two-rounds": [W.RowSpec(W.DECODE, 900, 1)] + 16 * CHUNK,
    "copied-past-them": [W.RowSpec(W.DECODE, 900, 1)] + 17 * CHUNK,
}


@pytest.mark.parametrize("name", list(CASES))
def test_plan_delivery(name):
    import torch
    from paper_2504_03651_amd.session import Iteration
    w = W.build(name, CASES[name], {}, 32, 32, 64, seed=101)
    say(f"[case] plan delivery {name}: rows={w.batch.num_rows}")
    it = Iteration(w)
    for _ in range(6):                    # round the ring of host buffers and past it
        it.out.fill_(float("nan"))
        it.step()
    torch.cuda.synchronize()
    _, ref = oracle.run_iteration(w)
    err, _ = attn_error(it.out.cpu().numpy().reshape(ref.shape), ref)
    say(f"       max abs err {err:.3e}")
    assert err <= ATOL


@pytest.mark.parametrize("slots", [1, 4])
def test_plans_that_follow_each_other(slots):
    # a buffer is rewritten with the next plan as soon as it is handed out again:
    # a kernel that read another call's plan would give that call's rows
    import torch
    from paper_2504_03651_amd import echo
    from paper_2504_03651_amd.session import Iteration
    order = ["direct-merge", "copied", "direct", "chunk-only", "copied-chunk", "direct-chunk",
             "direct-two-rounds", "copied-past-them"]
    its, refs = [], []
    for k, name in enumerate(order):
        rows = CASES[name][k % 2:] + CASES[name][:k % 2]    # in another order
        w = W.build(name, rows, {}, 32, 32, 64, seed=107 + k)
        it = Iteration(w)
        it.copy()
        it.append()
        its.append(it)
        refs.append(oracle.run_iteration(w)[1])
    # one workspace for all calls of the stream, sized for the largest
    ws = torch.empty(max(it.workspace.numel() for it in its), dtype=torch.uint8, device="cuda")
    hw = echo.HostWorkspace(slots=slots)
    outs = []
    torch.cuda.synchronize()
    say(f"[case] plans one after the other, {slots} buffers")
    for turn in range(3):
        for k in range(len(its)):
            it = its[(5 * k + turn) % len(its)]
            out = torch.full_like(it.out, float("nan"))
            echo.attn_mixed(it.pool, it.batch, it.q, 32, it.w.sm_scale, out, ws, host_workspace=hw)
            outs.append(((5 * k + turn) % len(its), out))
    torch.cuda.synchronize()
    for i, out in outs:
        err, _ = attn_error(out.cpu().numpy().reshape(refs[i].shape), refs[i])
        assert err <= ATOL, (order[i], err)
    hw.close()


@pytest.mark.parametrize("name", ["direct-merge", "copied-chunk"])
def test_captured_call_replays(name):
    import torch
    from paper_2504_03651_amd import echo
    from paper_2504_03651_amd.session import Iteration
    w = W.build(name, CASES[name], {}, 32, 32, 64, seed=103)
    say(f"[case] captured {name}")
    it = Iteration(w)
    it.step()
    torch.cuda.synchronize()
    want = it.out.clone()
    hw = echo.HostWorkspace(slots=1)
    ptr, size, _ = hw.acquire(echo.host_workspace_bytes(it.pool, it.batch, 32))
    cp, cb = it.pool.c(), it.batch.c()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rc = echo.lib().echo_attn_mixed(
            ctypes.byref(cp), ctypes.byref(cb), it.q.data_ptr(), 32, w.sm_scale, it.out.data_ptr(),
            it.workspace.data_ptr(), it.workspace.numel(), ptr, size,
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == echo.ECHO_OK, echo.last_error()
    for _ in range(4):
        it.out.fill_(float("nan"))
        it.workspace.fill_(0x5A)          # other work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(it.out.view(torch.int32), want.view(torch.int32))
    hw.close()
