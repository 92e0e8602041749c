"""The merge of partial states at the edges of its rounds: 64 slots per table round, 32 per element round.

The paged call writes one state per split of 64 blocks of the length bound, so the bound sets the slot count; one
beam fills every split, one leaves all but the first empty, one is empty.
"""

import math

import numpy as np
import pytest
import torch

from paper_2509_00195_amd import make_desc, tts_paged_decode_attn, tts_paged_decode_workspace_size

pytestmark = pytest.mark.gpu

POOL, G, HKV = 48, 3, 2


@pytest.mark.parametrize("kv,d,tol", [("bf16", 128, 1e-2), ("bf16", 64, 1e-2), ("f32", 128, 1e-4), ("f32", 64, 1e-4)])
@pytest.mark.parametrize("slots", [2, 31, 32, 33, 63, 64, 65, 97])
def test_merge_slot_counts(kv, d, tol, slots):
    g = torch.Generator().manual_seed(slots)
    dt = torch.float32 if kv == "f32" else torch.bfloat16
    bound = 1024 * slots
    lens = np.array([bound, 7, 0, bound - 1024 - 5], np.int32)
    tables = torch.randint(0, POOL, (len(lens), bound // 16), generator=g, dtype=torch.int32)
    q = torch.randn((len(lens), G * HKV, d), generator=g).to(dt)
    k = torch.randn((POOL, HKV, 16, d), generator=g).to(dt)
    v = torch.randn((POOL, HKV, d, 16), generator=g).to(dt)
    desc = make_desc(G * HKV, HKV, d, 16, kv, kv)
    nbytes = tts_paged_decode_workspace_size(desc, len(lens), bound)
    assert nbytes > 0
    out = torch.full((len(lens), G * HKV, d), float("nan"), device="cuda")
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")  # every float a NaN
    dev = [t.cuda() for t in (q, k, v, tables, torch.from_numpy(lens))]
    tts_paged_decode_attn(desc, len(lens), dev[0], dev[1], dev[2], None, None, dev[3], tables.shape[1], dev[4], bound,
                          POOL, out, ws, nbytes)
    got = out.cpu().double()
    for b, n in enumerate(lens):
        if n == 0:
            assert torch.all(got[b] == 0)
            continue
        ids = tables[b, : -(-int(n) // 16)].long()
        kk = k[ids].double().permute(1, 0, 2, 3).reshape(HKV, -1, d)[:, :n]
        vv = v[ids].double().permute(1, 0, 3, 2).reshape(HKV, -1, d)[:, :n]
        s = torch.matmul(q[b].double().reshape(HKV, G, d), kk.transpose(1, 2)) / math.sqrt(d)
        ref = torch.matmul(torch.softmax(s, -1), vv).reshape(G * HKV, d)
        assert float((got[b] - ref).abs().max()) <= tol, (b, int(n))
