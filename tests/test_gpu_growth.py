"""Beams that grew by different amounts since the metadata was built: their new blocks, packed over the beams of a unit
into windows of 64, against the oracle; a new block outside the pool makes that beam's rows NaN and no other's."""

import numpy as np
import pytest
import torch

from oracle.attention import oracle_attn_workload
from paper_2509_00195_amd import (
    tts_build_prefix_meta,
    tts_plan_units_host,
    tts_prefix_decode_attn,
    tts_prefix_decode_workspace_size,
)
from paper_2509_00195_amd.runner import desc_for
from paper_2509_00195_amd.tts import PLAN_SECOND
from tts_synth import AttnShape, ReqSpec, WorkloadConfig, make_workload
from tts_synth.device import to_device

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1e-2, "fp8": 2e-2, "f32": 1e-4}
GROWTHS = {
    "mixed": [0, 1, 15, 16, 17, 100, 1100, 333, 64],  # more than one window, some beams in two
    "few": [1, 0, 16, 0, 0, 33, 2, 0, 5],             # shares the first window
    "one": [0, 0, 0, 0, 1180, 0, 0, 0, 0],
    "all": [40] * 9,
}


@pytest.mark.parametrize("kv,d", [("bf16", 128), ("fp8", 128), ("f32", 64), ("bf16", 64)])
@pytest.mark.parametrize("prompt", [100, 16 * 9])
@pytest.mark.parametrize("name", sorted(GROWTHS))
def test_grown_beams(kv, d, prompt, name):
    shape = AttnShape(14, 2, d, 16, "f32" if kv == "f32" else "bf16", kv)
    spec = ReqSpec(beams=9, branch=1, prompt=(prompt, prompt), step=(1190, 1290), max_len=1 << 20, max_iters=1,
                   snapshot="none")
    wl = make_workload(WorkloadConfig("grown", shape, (spec,)), 3, shuffle=False)
    x = to_device(wl)
    desc = desc_for(shape)
    built = wl.seq_lens - np.array(GROWTHS[name], np.int32)
    # Only the blocks in use when the metadata is built are known then.
    tables = np.where(np.arange(wl.block_tables.shape[1])[None] < -(-built[:, None] // 16), wl.block_tables, -1)
    meta = tts_build_prefix_meta(wl.req_seq_offsets, tables, built, 16, wl.num_blocks, desc=desc)
    nbytes = tts_prefix_decode_workspace_size(desc, meta)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty((wl.num_seqs, 14, d), device="cuda")

    def run(tabs):
        tts_prefix_decode_attn(desc, meta, x.q, x.k_cache, x.v_cache, x.k_scale, x.v_scale, tabs, tabs.shape[1],
                               x.seq_lens, wl.num_blocks, out, ws, nbytes)
        return out.cpu().numpy()

    ref = oracle_attn_workload(wl)
    assert float(np.max(np.abs(run(x.block_tables) - ref))) <= TOL[kv]
    b = int(np.argmax(GROWTHS[name]))
    bad = x.block_tables.clone()
    bad[b, (int(wl.seq_lens[b]) - 1) // 16] = wl.num_blocks
    got = run(bad)
    rest = np.arange(wl.num_seqs) != b
    assert np.isnan(got[b]).all() and float(np.max(np.abs(got[rest] - ref[rest]))) <= TOL[kv]


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_grown_beams_of_units_with_two_windows(kv):
    """Units whose own entries fill two windows: what their beams gained comes after both."""
    shape = AttnShape(28, 4, 64, 16, "bf16", kv)
    spec = ReqSpec(beams=4, branch=1, prompt=(40, 40), step=(2100, 2400), max_len=1 << 20, max_iters=1, snapshot="none")
    wl = make_workload(WorkloadConfig("windows", shape, (spec,) * 96), 5)
    rng = np.random.default_rng(6)
    grown = np.where(rng.random(wl.num_seqs) < 0.5, rng.integers(0, 400, wl.num_seqs), 0).astype(np.int32)
    built = wl.seq_lens - grown
    tables = np.where(np.arange(wl.block_tables.shape[1])[None] < -(-built[:, None] // 16), wl.block_tables, -1)
    desc = desc_for(shape)
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    rows, _ = tts_plan_units_host(wl.req_seq_offsets, tables, built, 16, wl.num_blocks, desc, ncu)
    with_second = np.unique(rows[(rows[:, 6] & PLAN_SECOND) != 0, 0])
    beams = np.unique(rows[np.isin(rows[:, 0], with_second), 3])
    assert len(with_second) > 50 and (grown[beams] > 16).sum() > 20
    x = to_device(wl)
    meta = tts_build_prefix_meta(wl.req_seq_offsets, tables, built, 16, wl.num_blocks, desc=desc)
    nbytes = tts_prefix_decode_workspace_size(desc, meta)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty((wl.num_seqs, 28, 64), device="cuda")
    tts_prefix_decode_attn(desc, meta, x.q, x.k_cache, x.v_cache, x.k_scale, x.v_scale, x.block_tables,
                           x.block_tables.shape[1], x.seq_lens, wl.num_blocks, out, ws, nbytes)
    assert float(np.max(np.abs(out.cpu().numpy() - oracle_attn_workload(wl)))) <= TOL[kv]
