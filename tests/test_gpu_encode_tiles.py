"""Encodes at the edges of chunks (4096 values), bitmap bytes (8 blocks, shared
by several chunks above B = 512) and exception runs, against the CPU oracle
byte for byte: plain, with the fused cache update, with the block hash, and in
fp16."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    from paper_2609_04609_amd import ciera
    ciera.lib()
    return gpu_util


def check(gu, orc, n, B, c, seed):
    """Every encoder on one shard with change rate c (1.0: a cache that
    disagrees everywhere)."""
    from paper_2609_04609_amd import ciera, synth
    ws = ciera.Workspace(n, 1, B)
    w, w2 = gu.pair(n, seed, c=min(c, 0.5))
    w2h = gu.host_u16(w2)
    cache_h = orc.split(gu.host_u16(w))[0]
    if c == 1.0:
        cache_h = orc.split(w2h)[0] ^ 1
    msg = f"n={n} B={B} c={c}"
    expect = orc.encode(w2h, cache_h, B)
    out, total, _ = gu.gpu_encode(w2, gu.dev_u8(cache_h), B, ws)
    got = gu.host_u8(out)
    np.testing.assert_array_equal(got[:total], expect, err_msg=msg)
    assert (got[total:] == 0xA5).all(), msg
    gu.check_fused_update(orc, w2, cache_h, B, expect, ws, msg=msg)
    if B > 1 and c < 1.0:
        h = torch.empty(2 * ((n + B - 1) // B), dtype=torch.int64,
                        device="cuda")
        ciera.hash_blocks_t(w, B, h)
        np.testing.assert_array_equal(
            h.cpu().numpy().view(np.uint64).ravel(),
            orc.hash_blocks(gu.host_u16(w), B).ravel(), err_msg=msg)
        out.fill_(0xA5)
        ciera.encode_hashed_t(w2, h, h, B, ws, out)
        got = gu.host_u8(out)
        np.testing.assert_array_equal(got[:total], expect, err_msg=msg)
        np.testing.assert_array_equal(
            h.cpu().numpy().view(np.uint64).ravel(),
            orc.hash_blocks(w2h, B).ravel(), err_msg=msg)
    if B > 1:
        f = synth.normal_f16_bits(n, 0.02, seed + 5, "cuda")
        f2 = synth.forced_bernoulli_f16_bits(f, min(c, 0.5), seed + 6)
        fc = orc.split_f16(gu.host_u16(f))[0]
        expect = orc.encode_f16(gu.host_u16(f2), fc, B)
        fb = torch.full((int(ciera.ciera_encoded_bound(n, B, ciera.FP16)),),
                        0xA5, dtype=torch.uint8, device="cuda")
        ciera.encode_t(f2, gu.dev_u8(fc), B, ws, fb, fp16=True)
        got = gu.host_u8(fb)
        np.testing.assert_array_equal(got[:expect.size], expect, err_msg=msg)
        assert (got[expect.size:] == 0xA5).all(), msg
        gu.check_fused_update(orc, f2, fc, B, expect, ws, fp16=True, msg=msg)
    assert ws.error() == 0


@pytest.mark.parametrize("B", [1024, 2048, 4096])
@pytest.mark.parametrize("chunks", [33, 64, 65, 8 * 37 + 3])
def test_shared_bitmap_bytes(gu, orc, B, chunks):
    """A last bitmap byte that 1 ... 8 chunks share, and last chunks of one
    value, all but one, and all."""
    for i, tail in enumerate((-4095, -1, 0, 1 - B)):
        n = chunks * 4096 + tail
        for k, c in enumerate((0.0002, 1.0)):
            check(gu, orc, n, B, c, 7000 + 10 * chunks + 2 * i + k)


@pytest.mark.parametrize("B", [1, 16, 64, 512, 1024, 4096])
def test_small_shards(gu, orc, B):
    """The one-workgroup encode: no value, one octet and less, the edges of
    chunks and blocks, its largest shards (32,768 and 49,152 values) and
    the first ones that take two kernels."""
    for i, n in enumerate((0, 1, 7, 9, 4095, 4096, 4097, 8 * 4096 + 1,
                           49_151, 49_152, 49_153, 8 * 4096)):
        for k, c in enumerate((0.0, 0.003, 1.0)):
            check(gu, orc, n, B, c, 9000 + 100 * B + 3 * i + k)
