"""The work plan (host planner), on the CPU through tts_plan_units_host.

Properties that any correct plan has, checked on every workload shape at
several workgroup counts: for every KV head, each (beam, logical block) of
the build-time sequences is covered by exactly one unit entry, with the
block's physical id and valid token count from the block tables; the
partially filled last block of a beam is flagged LIVE and lies in a narrow
unit; every beam has exactly one extension entry per KV head (for blocks
appended after the build); LIVE and extension entries sit in a unit's first
window; a window holds at most 64 entries (a unit at most 128); wide units
hold full blocks only. The number of units bounds the partial states.
"""

import dataclasses

import numpy as np
import pytest

import paper_2509_00195_amd as tts
from paper_2509_00195_amd.tts import PLAN_EXT, PLAN_LIVE, PLAN_SECOND, PLAN_WIDE
from tts_synth import CONFIGS, AttnShape, ReqSpec, WorkloadConfig, build_tree, workload_from_tree

BS = 16


def tables_of(cfg, seed):
    """The config's beam tree, block tables and lengths (the plan needs no cache contents: tiny values)."""
    return workload_from_tree(AttnShape(2, 1, 8, BS, "f32", "f32"), build_tree(cfg, seed), seed, name=cfg.name)


def plan_rows(wl, sh, nbins):
    desc = tts.make_desc(sh.num_q_heads, sh.num_kv_heads, sh.head_dim, BS, sh.q_dtype, sh.kv_dtype)
    return tts.tts_plan_units_host(wl.req_seq_offsets, wl.block_tables, wl.seq_lens, BS, wl.num_blocks, desc, nbins)


def check_plan(wl, sh, nbins):
    rows, units = plan_rows(wl, sh, nbins)
    unit, entry, kvh, beam, block, valid, flags = rows.T
    assert units >= 1 and unit.min() == 0 and unit.max() == units - 1
    ext = (flags & PLAN_EXT) != 0
    # coverage: exactly once per (kv head, beam, logical block)
    lens = np.asarray(wl.seq_lens, np.int64)
    tabs = np.asarray(wl.block_tables, np.int64)
    nblk = (lens + BS - 1) // BS
    pos = {}
    for b in range(len(lens)):
        for j in range(int(nblk[b])):
            pos[(b, int(tabs[b, j]))] = j
    seen = np.zeros((sh.num_kv_heads, len(lens), int(nblk.max()) if len(lens) else 0), np.int32)
    for u, h, b, blk, v, f in zip(unit[~ext], kvh[~ext], beam[~ext], block[~ext], valid[~ext], flags[~ext]):
        j = pos[(int(b), int(blk))]
        seen[h, b, j] += 1
        assert v == min(BS, int(lens[b]) - BS * j)
        partial = j == nblk[b] - 1 and lens[b] % BS != 0
        assert bool(f & PLAN_LIVE) == partial
        if f & PLAN_WIDE:
            assert v == BS and not partial
    for b in range(len(lens)):
        assert (seen[:, b, : nblk[b]] == 1).all(), b
    # one extension entry per (kv head, beam)
    ext_count = np.zeros((sh.num_kv_heads, len(lens)), np.int32)
    np.add.at(ext_count, (kvh[ext], beam[ext]), 1)
    assert (ext_count == 1).all()
    # windows
    assert not ((flags & (PLAN_LIVE | PLAN_EXT)) != 0)[(flags & PLAN_SECOND) != 0].any()
    for w in (0, PLAN_SECOND):
        sel = (flags & PLAN_SECOND) == w
        per_window = {}
        for u, e in zip(unit[sel], entry[sel]):
            per_window.setdefault(int(u), set()).add(int(e))
        assert all(len(es) <= 64 for es in per_window.values())
    return rows, units


@pytest.mark.parametrize("name", ["tiny", "1p5b16", "7b64", "7b64_balanced", "7b_straggler"])
@pytest.mark.parametrize("seed", [0, 1])
@pytest.mark.parametrize("nbins", [256, 40, 1])
def test_plan_covers_every_block_once(name, seed, nbins):
    cfg = CONFIGS[name]
    check_plan(tables_of(cfg, seed), cfg.shape, nbins)


def test_long_chain_plan_uses_both_windows():
    cfg = CONFIGS["7b_longchain_fp8"]
    cfg = dataclasses.replace(cfg, reqs=cfg.reqs[:4])  # a quarter of the requests keeps the check quick
    rows, units = check_plan(tables_of(cfg, 0), cfg.shape, 64)
    flags = rows[:, 6]
    assert ((flags & PLAN_SECOND) != 0).any() and ((flags & PLAN_WIDE) != 0).any()


def test_small_batch_gets_few_units():
    """A batch that fits the workgroups gets units sized by attention plus merge time, not one per entry:
    at most a few units per beam and KV head."""
    cfg = CONFIGS["1p5b16"]
    for seed in range(6):
        wl = tables_of(cfg, seed)
        _, units = plan_rows(wl, cfg.shape, 256)
        assert units <= 4 * len(wl.seq_lens) * cfg.shape.num_kv_heads, (seed, units)


def test_plan_argument_errors():
    sh = CONFIGS["tiny"].shape
    wl = tables_of(CONFIGS["tiny"], 0)
    desc = tts.make_desc(sh.num_q_heads, sh.num_kv_heads, sh.head_dim, BS, sh.q_dtype, sh.kv_dtype)
    with pytest.raises(tts.TTSError):
        tts.tts_plan_units_host(wl.req_seq_offsets, wl.block_tables, wl.seq_lens, BS, wl.num_blocks, desc, 0)
    bad = np.where(wl.block_tables == wl.block_tables[0, 0], wl.num_blocks + 5, wl.block_tables).astype(np.int32)
    with pytest.raises(tts.TTSError):
        tts.tts_plan_units_host(wl.req_seq_offsets, bad, wl.seq_lens, BS, wl.num_blocks, desc, 8)


def unit_rows(name, wide, nbins=256):
    """Query rows of each wide (or each narrow) unit in the seed-0 plan of a config."""
    cfg = CONFIGS[name]
    rows, _ = plan_rows(tables_of(cfg, 0), cfg.shape, nbins)
    unit, beam, flags = rows[:, 0], rows[:, 3], rows[:, 6]
    sel = ((flags & PLAN_WIDE) != 0) == wide
    g = cfg.shape.num_q_heads // cfg.shape.num_kv_heads
    beams = {}
    for u, b in zip(unit[sel], beam[sel]):
        beams.setdefault(int(u), set()).add(int(b))
    return [g * len(v) for v in beams.values()]


def test_row_caps_are_chosen_per_batch():
    """A batch of much KV per workgroup takes wide units of up to 128 rows (one row tile per wave) and narrow ones of
    up to 32, others of up to 192 (two tiles) and 64, or 256-row wide units where these model faster: 192 / 64 for
    the 7B 64-beam tree, 128 for the balanced tree; the 1.5B 16-beam tree's narrow units stay within 42 rows."""
    r = unit_rows("7b64", wide=True)
    assert r and 128 < max(r) <= 192
    assert 42 < max(unit_rows("7b64", wide=False)) <= 64
    r = unit_rows("7b64_balanced", wide=True)
    assert r and max(r) <= 128
    assert max(unit_rows("1p5b16", wide=False)) <= 42


def test_states_fit_the_scratch_array():
    """A batch of 3072 beams whose plan of the fastest units writes more than the 64 MiB of partial states that the
    allocation-free call holds: the plan taken writes less. (Shared segments of 33 to 64 rows are units of their own
    in the fastest plan, one more state for each of their beams.)"""
    reqs, beams, g, hkv, d = 48, 64, 7, 4, 128
    nxt = 0
    tables = np.full((reqs * beams, 64), -1, np.int32)
    lens = np.zeros(reqs * beams, np.int32)

    def fresh(n):
        nonlocal nxt
        nxt += n
        return list(range(nxt - n, nxt))

    for r in range(reqs):  # a prompt, groups of 8 beams, pairs, private blocks
        prompt = fresh(12)
        for a in range(beams // 8):
            mid = fresh(5)
            for p in range(4):
                pair = fresh(4)
                for k in range(2):
                    b = r * beams + a * 8 + p * 2 + k
                    ids = prompt + mid + pair + fresh(3)
                    tables[b, : len(ids)] = ids
                    lens[b] = 16 * len(ids) - 5
    offs = np.arange(reqs + 1, dtype=np.int32) * beams
    desc = tts.make_desc(g * hkv, hkv, d, BS, "bf16", "bf16")
    rows, _ = tts.tts_plan_units_host(offs, tables, lens, BS, nxt, desc, 256)
    own = rows[rows[:, 2] == 0]
    states = len(np.unique(own[:, 0].astype(np.int64) * len(lens) + own[:, 3]))
    assert states * g * hkv * (2 * d + 16) <= 64 << 20


@pytest.mark.parametrize("name", ["1p5b16", "7b64", "7b64_balanced"])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_plan_covers_every_block_once(name, d):
    check_plan(tables_of(CONFIGS[name], 0), AttnShape(28, 4, d, BS, "f32", "f32"), 256)


def test_fp32_segments_take_full_units_in_a_streaming_batch():
    """fp32 caches have no wide units: a long segment of many beams is cut into narrow-mode units of up to 64 rows,
    each of which reads its blocks again, also where the batch's private tails are listed in units of fewer rows."""
    reqs, beams, shared, tail = 4, 63, 450, 3
    tables = np.zeros((reqs * beams, shared + tail), np.int32)
    nxt = 0
    for r in range(reqs):
        tables[r * beams:(r + 1) * beams, :shared] = nxt + np.arange(shared)
        nxt += shared
        for b in range(r * beams, (r + 1) * beams):
            tables[b, shared:] = nxt + np.arange(tail)
            nxt += tail
    lens = np.full(reqs * beams, 16 * (shared + tail), np.int32)
    desc = tts.make_desc(28, 4, 128, BS, "f32", "f32")
    rows, _ = tts.tts_plan_units_host(np.arange(reqs + 1, dtype=np.int32) * beams, tables, lens, BS, nxt, desc, 256)
    of_shared = rows[(rows[:, 2] == 0) & np.isin(rows[:, 4], tables[:, :shared].ravel())]
    units = {u: 7 * len(set(of_shared[of_shared[:, 0] == u, 3].tolist())) for u in set(of_shared[:, 0].tolist())}
    assert units and min(units.values()) > 32 and max(units.values()) <= 64


@pytest.mark.parametrize("kv,hq,hkv,beams", [("fp8", 12, 2, 16), ("bf16", 12, 2, 16), ("bf16", 32, 8, 4)])
@pytest.mark.parametrize("cap", [4096, 12000])
def test_long_tails_of_few_beams_fill_the_workgroups_once(kv, hq, hkv, beams, cap):
    """Few beams with long private tails: the tails are cut so that the workgroups get about one unit each, however
    many states that leaves per beam (not half of them, nor three each)."""
    spec = ReqSpec(beams=beams, branch=4, prompt=(300, 300), step=(64, 256), max_len=cap, rule="balanced")
    sh = AttnShape(hq, hkv, 128, BS, "bf16", kv)
    _, units = plan_rows(tables_of(WorkloadConfig("tails", sh, (spec,)), 0), sh, 256)
    assert 192 <= units <= 256


def test_many_small_requests_are_units_of_their_own():
    """Hundreds of requests of eight beams with short prompts and tails: chained by the dozen, units have to be few. A
    request (56 rows of one KV head) is about one unit, not one for its prompt and one for every four beams' tails."""
    reqs, beams, prompt, tail = 240, 8, 5, 4
    tables = np.zeros((reqs * beams, prompt + tail), np.int32)
    nxt = 0
    for r in range(reqs):
        for b in range(r * beams, (r + 1) * beams):
            tables[b, :prompt] = nxt + np.arange(prompt)
            tables[b, prompt:] = nxt + prompt + (b - r * beams) * tail + np.arange(tail)
        nxt += prompt + beams * tail
    lens = np.full(reqs * beams, 16 * (prompt + tail) - 3, np.int32)
    desc = tts.make_desc(28, 4, 128, BS, "bf16", "bf16")
    _, units = tts.tts_plan_units_host(np.arange(reqs + 1, dtype=np.int32) * beams, tables, lens, BS, nxt, desc, 256)
    assert units <= 1.5 * reqs * 4
