"""Calls of more than 2^32 threads, which no launch holds: made in runs of whole beams.

The paged call (48 GB) is beyond one launch in both of its kernels: 17 query heads per KV head take several row tiles,
512 threads per workgroup, and two splits per beam, so the attention of 4,194,308 beams has 8,388,616 workgroups
(8,388,607 fit) and the merge 71 million rows (67 million fit). Nearly all beams are empty; those at the ends of the
runs are not. The append has two workgroups of 256 threads per beam (8,388,607 beams fit).
"""

import math

import pytest
import torch

from paper_2509_00195_amd import make_desc, tts_append_kv, tts_paged_decode_attn, tts_paged_decode_workspace_size

pytestmark = pytest.mark.gpu

G, D, POOL, BOUND = 17, 64, 40, 513
ATTN_RUN = (2 ** 32 - 1) // 512 // 8 * 8 // 2        # beams of an attention launch
MERGE_RUN = (2 ** 32 - 1) // 256 * 4 // G            # beams of a merge launch


def test_call_of_more_threads_than_a_launch_holds():
    n = ATTN_RUN + 8
    assert n * G > (2 ** 32 - 1) // 64
    picks = sorted({0, 1, MERGE_RUN - 1, MERGE_RUN, MERGE_RUN + 1, ATTN_RUN - 1, ATTN_RUN, ATTN_RUN + 1, n - 1})
    gen = torch.Generator().manual_seed(0)
    cols = -(-BOUND // 16)
    lens = torch.zeros(n, dtype=torch.int32, device="cuda")
    tables = torch.zeros((n, cols), dtype=torch.int32, device="cuda")
    q = torch.zeros((n, G, D), dtype=torch.bfloat16, device="cuda")
    k = torch.randn((POOL, 1, 16, D), generator=gen).bfloat16()
    v = torch.randn((POOL, 1, D, 16), generator=gen).bfloat16()
    want = {}
    for i, b in enumerate(picks):
        length = (BOUND, 77, 512)[i % 3]
        tab = torch.randint(0, POOL, (cols,), generator=gen, dtype=torch.int32)
        qb = torch.randn((G, D), generator=gen).bfloat16()
        lens[b], tables[b], q[b] = length, tab.cuda(), qb.cuda()
        ids = tab[: -(-length // 16)].long()
        kk = k[ids, 0].double().reshape(-1, D)[:length]
        vv = v[ids, 0].double().transpose(1, 2).reshape(-1, D)[:length]
        want[b] = torch.matmul(torch.softmax(torch.matmul(qb.double(), kk.T) / math.sqrt(D), -1), vv)
    desc = make_desc(G, 1, D, 16, "bf16", "bf16")
    nbytes = tts_paged_decode_workspace_size(desc, n, BOUND)
    out = torch.full((n, G, D), float("nan"), device="cuda")
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")  # every float a NaN
    tts_paged_decode_attn(desc, n, q, k.cuda(), v.cuda(), None, None, tables, cols, lens, BOUND, POOL, out, ws, nbytes)
    for b in picks:
        assert float((out[b].cpu().double() - want[b]).abs().max()) <= 1e-2, b
        out[b] = 0
    for at in range(0, n, 1 << 18):  # the empty beams: zero rows
        assert int(torch.count_nonzero(out[at:at + (1 << 18)])) == 0, at
    del out, ws, q, tables
    torch.cuda.empty_cache()


def test_append_of_more_beams_than_a_launch_holds():
    run = (2 ** 32 - 1) // 512
    n = run + 3
    picks = torch.tensor([0, 1, run - 1, run, run + 1, n - 1], device="cuda")
    lens = torch.zeros(n, dtype=torch.int32, device="cuda")
    tables = torch.zeros((n, 1), dtype=torch.int32, device="cuda")
    lens[picks] = 5
    tables[picks, 0] = torch.arange(len(picks), dtype=torch.int32, device="cuda")
    k_new, v_new = (torch.randn((n, 1, D), device="cuda").bfloat16() for _ in range(2))
    k = torch.zeros((len(picks), 1, 16, D), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros((len(picks), 1, D, 16), dtype=torch.bfloat16, device="cuda")
    tts_append_kv(make_desc(G, 1, D, 16, "bf16", "bf16"), n, k_new, v_new, tables, 1, lens, len(picks), k, v, None, None)
    assert torch.equal(k[:, :, 4], k_new[picks]) and torch.equal(v[..., 4], v_new[picks])
    k[:, :, 4] = 0
    v[..., 4] = 0
    assert int(torch.count_nonzero(k)) == int(torch.count_nonzero(v)) == 0
