"""The merge of partial states at the edges of its rounds: 64 slots per table round, 32 per element round.

The paged call writes one state per split of 32 blocks of the length bound, so the bound sets the slot count; one beam
fills every split, one leaves all but the first empty, one is empty, one leaves the last empty.

Every split's state is exact: its scores are one integer in log2 units, its values one small integer per dimension, so
probabilities (powers of two), sums and stored elements carry no rounding, and the result is off by that of the merge
alone, in fp32. A dropped, repeated or exchanged slot moves it far more, which the test checks of every slot.
"""

import math

import numpy as np
import pytest
import torch

from oracle.attention import oracle_attn_workload
from paper_2509_00195_amd import make_desc, tts_paged_decode_attn, tts_paged_decode_workspace_size, tts_prefix_meta_stats
from paper_2509_00195_amd.runner import PrefixAttention
from tts_synth import AttnShape, ReqSpec, WorkloadConfig, make_workload
from tts_synth.device import to_device

pytestmark = pytest.mark.gpu

G, HKV, SPLIT, VMAX = 3, 2, 512, 8


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("slots", [2, 31, 32, 33, 63, 64, 65, 96, 97, 129])
def test_merge_slot_counts(kv, d, slots):
    g = torch.Generator().manual_seed(slots)
    dt = torch.float32 if kv == "f32" else torch.bfloat16
    bound = SPLIT * slots
    # A stored element is (tokens x value) / 2^e in fp16, exact while that product has 11 bits: 512 v, 7 v, 8 x 63 v.
    lens = np.array([bound, 7, 0, bound - SPLIT - 8], np.int32)
    order = torch.randperm(slots, generator=g)  # split j: 32 times block order[j]
    tables = order.to(torch.int32).repeat_interleave(SPLIT // 16).expand(len(lens), -1).contiguous()
    score = torch.randint(-3, 4, (slots, HKV), generator=g)
    value = torch.randint(-VMAX, VMAX + 1, (slots, HKV, d), generator=g)
    k = torch.zeros((slots, HKV, 16, d), dtype=dt)
    k[order, :, :, 0] = score[:, :, None].to(dt)
    v = torch.zeros((slots, HKV, d, 16), dtype=dt)
    v[order] = value[..., None].to(dt)
    sign = torch.tensor([1, -1, 0]).repeat(HKV)  # heads with weights 2^score, 2^-score and 1
    q = torch.zeros((len(lens), G * HKV, d), dtype=dt)
    q[:, :, 0] = sign.to(dt)
    desc = make_desc(G * HKV, HKV, d, 16, kv, kv, "f32", math.log(2.0))
    nbytes = tts_paged_decode_workspace_size(desc, len(lens), bound)
    rows = len(lens) * slots * G * HKV
    assert nbytes == sum(-(-rows * n // 256) * 256 for n in (d * (4 if kv == "f32" else 2), 16))
    out = torch.full((len(lens), G * HKV, d), float("nan"), device="cuda")
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")  # every float a NaN
    dev = [t.cuda() for t in (q, k, v, tables, torch.from_numpy(lens))]
    tts_paged_decode_attn(desc, len(lens), dev[0], dev[1], dev[2], None, None, dev[3], tables.shape[1], dev[4], bound,
                          slots, out, ws, nbytes)
    got = out.cpu().double()
    # slots + 8 roundings of sums and products, each at most 2^-23 of the largest value
    tol = (slots + 8) * 2.0 ** -23 * VMAX
    kvh = torch.arange(G * HKV) // G
    val = value[:, kvh].double()  # [slots][heads][d]
    for b, n in enumerate(lens):
        if n == 0:
            assert torch.all(got[b] == 0)
            continue
        tokens = (int(n) - SPLIT * torch.arange(slots)).clamp(0, SPLIT).double()
        w = tokens[:, None] * 2.0 ** (score[:, kvh] * sign)
        total, den = (w[..., None] * val).sum(0), w.sum(0)[:, None]
        ref = total / den
        assert float((got[b] - ref).abs().max()) <= tol, (b, int(n))
        used = int((tokens > 0).sum())
        for j in range(used if used > 1 else 0):
            for times in (-1, 1):  # without slot j, and with it twice
                moved = (total + times * w[j][:, None] * val[j]) / (den + times * w[j][:, None])
                assert float((moved - ref).abs().max()) > 20 * tol, (b, j)


@pytest.mark.parametrize("d", [64, 128])
def test_merge_of_a_long_beam_through_the_slot_table(d):
    """A beam alone on the GPU is split over most workgroups: more slots than the table round reads ahead (64). fp32,
    where leaving out a slot moves the result by more than the tolerance."""
    spec = ReqSpec(beams=1, branch=1, prompt=(60000, 60000), step=(7, 7), max_len=1 << 20, max_iters=1, snapshot="none")
    wl = make_workload(WorkloadConfig("long", AttnShape(2, 1, d, 16, "f32", "f32"), (spec,)), 1)
    pref = PrefixAttention(to_device(wl), wl.req_seq_offsets, wl.block_tables, wl.seq_lens, wl.num_blocks)
    _, slots = tts_prefix_meta_stats(pref.meta)
    assert slots > 96  # of the one beam
    pref.ws.fill_(255)  # every float a NaN
    ref = oracle_attn_workload(wl)
    assert float(np.max(np.abs(pref().cpu().numpy() - ref))) <= 2e-6 + 1e-5 * float(np.max(np.abs(ref)))
