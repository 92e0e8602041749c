"""The paged call at the edges of a unit: 1 to 16 query heads per KV head in one row tile and more in several, lengths
around a block, a pair of blocks, a round of pairs of four waves and a split, unit counts that are no multiple of 8."""

import math

import numpy as np
import pytest
import torch

from paper_2509_00195_amd import make_desc, tts_paged_decode_attn, tts_paged_decode_workspace_size

pytestmark = pytest.mark.gpu

POOL, HKV = 40, 3
# A split takes 512 tokens at the bounds 1024 and 2500 and 368 at 1100.
LENS = (1, 16, 17, 32, 33, 128, 129, 0, 367, 368, 369, 511, 512, 513, 700, 1023, 1024, 1025, 1100)


def tolerance(kv, v):
    """fp32 caches: the attention calls' parity tolerance. Else the probabilities (times the value scales) are rounded
    to bf16 for the value product and their sum is not, so a row is off by at most 2^-8 sum(p |v|) / sum(p), and a
    split's state is stored in fp16, at most 2^-11 of its largest element more: with |v| at most max, whatever the
    length, 2^-8 + 2^-11 of max (and 1e-5 for the fp32 sums)."""
    return 1e-4 if kv == "f32" else (2.0 ** -8 + 2.0 ** -11) * float(v.abs().max()) + 1e-5


@pytest.mark.parametrize("kv", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g,bound", [(1, 1024), (7, 1100), (15, 1024), (16, 2500), (17, 1100)])
def test_paged_units(kv, d, g, bound):
    gen = torch.Generator().manual_seed(g + d)
    lens = np.array([n for n in LENS if n <= bound], np.int32)
    nb = -(-lens // 16)
    cols = -(-bound // 16)
    tables = torch.randint(0, POOL, (len(lens), cols), generator=gen, dtype=torch.int32)
    for b in range(len(lens)):
        tables[b, nb[b]:] = -1  # past the length: must not matter
    bad = len(lens) - 1
    tables[bad, nb[bad] - 1] = POOL  # outside the pool: only this beam's rows
    q = torch.randn((len(lens), g * HKV, d), generator=gen).to(torch.float32 if kv == "f32" else torch.bfloat16)
    k = torch.randn((POOL, HKV, 16, d), generator=gen)
    v = torch.randn((POOL, HKV, d, 16), generator=gen)
    ks = torch.rand(POOL, generator=gen) + 0.5
    vs = torch.rand(POOL, generator=gen) + 0.5
    if kv == "fp8":
        k, v = k.to(torch.float8_e4m3fn), v.to(torch.float8_e4m3fn)
        k64 = k.double() * ks.double().reshape(-1, 1, 1, 1)
        v64 = v.double() * vs.double().reshape(-1, 1, 1, 1)
        k, v = k.view(torch.uint8), v.view(torch.uint8)
    else:
        dt = torch.float32 if kv == "f32" else torch.bfloat16
        k, v = k.to(dt), v.to(dt)
        k64, v64 = k.double(), v.double()
    desc = make_desc(g * HKV, HKV, d, 16, "f32" if kv == "f32" else "bf16", kv)
    nbytes = tts_paged_decode_workspace_size(desc, len(lens), bound)
    out = torch.full((len(lens), g * HKV, d), 7.0, device="cuda")
    ws = torch.full((max(nbytes, 1),), 255, dtype=torch.uint8, device="cuda")  # every float a NaN
    dev = [t.cuda() for t in (q, k, v, tables, torch.from_numpy(lens), ks, vs)]
    scales = (dev[5], dev[6]) if kv == "fp8" else (None, None)
    tts_paged_decode_attn(desc, len(lens), dev[0], dev[1], dev[2], *scales, dev[3], cols, dev[4], bound, POOL, out, ws,
                          nbytes)
    got = out.cpu().double()
    assert torch.isnan(got[bad]).all()
    for b, n in enumerate(lens[:bad]):
        if n == 0:
            assert torch.all(got[b] == 0)
            continue
        ids = tables[b, : nb[b]].long()
        kk = k64[ids].permute(1, 0, 2, 3).reshape(HKV, -1, d)[:, :n]
        vv = v64[ids].permute(1, 0, 3, 2).reshape(HKV, -1, d)[:, :n]
        s = torch.matmul(q[b].double().reshape(HKV, g, d), kk.transpose(1, 2)) / math.sqrt(d)
        ref = torch.matmul(torch.softmax(s, -1), vv).reshape(g * HKV, d)
        assert float((got[b] - ref).abs().max()) <= tolerance(kv, v64), (b, int(n))
