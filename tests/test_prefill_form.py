"""Which prefill form a call gets at head_dim 64 (CPU): two workgroups per CU by
the work there is, not by the size of a descriptor region, and only while two fit
the LDS.  The rule is compiled from
the planner's header; what the host planner makes of it shows in the order of its
prefill descriptors, longest first where two workgroups share a CU."""
import shutil
import subprocess

import numpy as np
import pytest

from paper_2504_03651_amd import build, echo
from paper_2504_03651_amd import workload as W

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "plan.hpp"
using namespace echo;
int main(int n, char **v) {   // tokens, rows, tokens per tile, KV heads, most blocks
    const int64_t t = prefill_tiles_at_least(atol(v[1]), atol(v[2]), atol(v[3]));
    printf("%d", prefill_two_per_cu(64, t * atol(v[4]), atol(v[5]), 256) ? 1 : 0);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_device_plans_go_by_the_tiles_that_have_work(tmp_path):
    src, exe = tmp_path / "form.cpp", str(tmp_path / "form")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, "-o", exe, str(src)], check=True)

    def form(tokens, rows, blocks=300):   # GQA 64/8: tiles of 32 tokens
        return subprocess.run([exe, *map(str, (tokens, rows, 32, 8, blocks))], check=True,
                              capture_output=True, text=True).stdout == "1"

    assert not form(64 + 500, 65)          # 128 workgroups, a region for 664
    assert not form(64 + 100, 65)
    assert not form(300, 300)              # decode rows alone
    assert form(9924, 12)                  # fresh prompts
    assert form(64 + 2200, 65)
    assert not form(9924, 12, 8001)        # block ids of 128,016 keys: one per CU


def _order(rows, hq, hkv):
    w = W.build("form", rows, {}, hq, hkv, 64, seed=1, values=False)
    cp, cb, _keep = echo.host_structs(w)
    lay, words = echo.plan_pack(cp, cb, hq)
    d = words[lay["off_pdesc"]:lay["off_pdesc"] + 8 * lay["n_pdesc"]].reshape(-1, 8)
    return d[:, 0], d[:, 3]


@pytest.mark.parametrize("ctx,hq,hkv,n,dense", [
    (0, 16, 16, 12, True),       # 528 workgroups
    (0, 64, 8, 23, True),
    (0, 64, 8, 19, False),       # 440
    (130000, 64, 8, 23, False),  # the ids of 8,130 blocks leave room for one per CU
])
def test_host_plans_sort_where_two_share_a_cu(ctx, hq, hkv, n, dense):
    tokens = 256 // (hq // hkv)
    rows = [W.RowSpec(W.PREFILL, ctx if i else 0, tokens * (1 + i % 5)) for i in range(n)]
    row, keys = _order(rows, hq, hkv)
    by_row = bool((np.diff(row) >= 0).all())
    assert by_row == (not dense)
    if dense:
        assert keys[0] == keys.max() and keys[-1] < keys[0]
