"""Append and block copies at the edges of their work split, bit-exact against the oracle: every slot of a block, tokens
of less and of more values than a workgroup's threads hold, caches that start at odd addresses, blocks of less than one
copied piece and of several with a remainder."""

import numpy as np
import pytest
import torch

from oracle.kv_ops import append_kv, copy_blocks
from paper_2509_00195_amd import make_desc, tts_append_kv, tts_copy_blocks

pytestmark = pytest.mark.gpu


def bits(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


def place(a, odd):
    """The array on the GPU, `odd` elements into a larger buffer."""
    flat = torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).reshape(-1).cuda()
    buf = torch.zeros(flat.numel() + odd, dtype=flat.dtype, device="cuda")
    buf[odd:] = flat
    return buf[odd:]


def host(t, like):
    return t.cpu().numpy().view(like.dtype).reshape(like.shape)


def cache(kv, nb, hkv, d, rng):
    if kv == "bf16":
        return bits(rng.normal(0, 1, (nb, hkv, 16, d))), bits(rng.normal(0, 1, (nb, hkv, d, 16))), None, None
    k, v = (rng.integers(0, 256, s, dtype=np.uint8) for s in ((nb, hkv, 16, d), (nb, hkv, d, 16)))
    for x in (k, v):
        x[(x & 0x7F) == 0x7F] = 0
    ks, vs = (np.full(nb, 0.005, np.float32) for _ in range(2))
    return k, v, ks, vs


SHAPES = [(1, 64), (3, 64), (4, 128), (10, 128)]


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("hkv,d", SHAPES)
@pytest.mark.parametrize("odd", [0, 1])
def test_append_every_slot(kv, hkv, d, odd):
    rng = np.random.default_rng(hkv * d + odd)
    s, nb = 34, 40
    k, v, ks, vs = cache(kv, nb, hkv, d, rng)
    tables = rng.permutation(nb)[:s].astype(np.int32)[:, None]
    lens = np.array([1 + i % 16 for i in range(s - 2)] + [0, 17], np.int32)  # the last: past its table row
    boost = np.where(np.arange(s) < 16, 1.0, 30.0)[:, None, None]  # the second sixteen raise their block's scale
    kn, vn = (bits(rng.normal(0, 1, (s, hkv, d)) * boost) for _ in range(2))
    desc = make_desc(2 * hkv, hkv, d, q_dtype="bf16", kv_dtype=kv)
    dk, dv = place(k, odd), place(v, odd)
    dks, dvs = (None if x is None else torch.from_numpy(x.copy()).cuda() for x in (ks, vs))
    dev = [place(x, 0) for x in (kn, vn, tables, lens)]
    tts_append_kv(desc, s, dev[0], dev[1], dev[2], 1, dev[3], nb, dk, dv, dks, dvs)
    append_kv(kv, k, v, ks, vs, tables, lens, kn, vn)
    assert np.array_equal(host(dk, k), k) and np.array_equal(host(dv, v), v)
    if ks is not None:
        assert np.array_equal(dks.cpu().numpy().view(np.uint32), ks.view(np.uint32))
        assert np.array_equal(dvs.cpu().numpy().view(np.uint32), vs.view(np.uint32))


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("hkv,d", SHAPES)
def test_copy_pieces(kv, hkv, d):
    rng = np.random.default_rng(hkv * d)
    nb = 24
    k, v, ks, vs = cache(kv, nb, hkv, d, rng)
    pairs = np.array([[0, 20], [1, 21], [1, 22], [23, 3], [4, 4], [nb, 5], [6, -1]], np.int32)
    if ks is not None:
        ks[:], vs[:] = rng.uniform(0.1, 1, (2, nb)).astype(np.float32)
    dk, dv = place(k, 0), place(v, 0)
    dks, dvs = (None if x is None else torch.from_numpy(x.copy()).cuda() for x in (ks, vs))
    tts_copy_blocks(make_desc(2 * hkv, hkv, d, q_dtype="bf16", kv_dtype=kv), len(pairs), place(pairs, 0), nb, dk, dv,
                    dks, dvs)
    copy_blocks(k, v, ks, vs, pairs)
    assert np.array_equal(host(dk, k), k) and np.array_equal(host(dv, v), v)
    if ks is not None:
        assert np.array_equal(dks.cpu().numpy(), ks) and np.array_equal(dvs.cpu().numpy(), vs)
