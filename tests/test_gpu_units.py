"""Units at the edges of their row tiles and wave groups: from one beam to more than a wide unit takes.

Rows of a unit are (beam, query head of the group). A shared prompt of an odd number of blocks gives wide units of up
to eight tiles (the workgroup's halves take alternate pairs) and of more (every wave takes every pair), with and
without a last half step; private tails give narrow units of one and of two wave groups (fp32: up to four).
"""

import numpy as np
import pytest

from oracle.attention import oracle_attn_workload
from paper_2509_00195_amd.runner import PagedAttention, PrefixAttention
from tts_synth import AttnShape, ReqSpec, WorkloadConfig, make_workload
from tts_synth.device import to_device

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1e-2, "fp8": 2e-2, "f32": 1e-4}


def check(shape, beams, prompt, seed=0):
    spec = ReqSpec(beams=beams, branch=1, prompt=(prompt, prompt), step=(1, 70), max_len=1 << 20, max_iters=1,
                   snapshot="none")
    wl = make_workload(WorkloadConfig("units", shape, (spec,)), seed)
    x = to_device(wl)
    ref = oracle_attn_workload(wl)
    pref = PrefixAttention(x, wl.req_seq_offsets, wl.block_tables, wl.seq_lens, wl.num_blocks)
    pref.ws.fill_(255)  # every partial state a NaN until it is written
    for call in (pref, PagedAttention(x, wl.max_seq_len, wl.num_blocks)):
        e = float(np.max(np.abs(call().cpu().numpy() - ref)))
        assert e <= TOL[shape.kv_dtype], (type(call).__name__, e)


@pytest.mark.parametrize("kv", ["bf16", "fp8", "f32"])
@pytest.mark.parametrize("beams", [1, 2, 3, 4, 5, 9, 10, 16, 18, 19, 36, 37])
def test_rows_of_seven_heads(kv, beams):
    check(AttnShape(14, 2, 128, 16, "f32" if kv == "f32" else "bf16", kv), beams, 16 * 21 + 9)


@pytest.mark.parametrize("kv", ["bf16", "fp8", "f32"])
@pytest.mark.parametrize("group,beams", [(16, 9), (17, 2), (33, 3), (48, 1), (64, 5)])
def test_large_head_groups(kv, group, beams):
    check(AttnShape(group, 1, 64, 16, "f32" if kv == "f32" else "bf16", kv), beams, 16 * 12 + 1)
