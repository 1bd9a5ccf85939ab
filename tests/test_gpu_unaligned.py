"""Buffers at any address: weights, caches and decoded values as slices that
start at odd places (shards whose length is no multiple of 8 put every later
shard there), through the whole-octet vector accesses. Byte for byte against
the CPU oracle, and no byte outside the slices may change."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 64  # values or bytes kept free around each slice


@pytest.fixture(scope="module")
def gu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    from paper_2609_04609_amd import ciera
    ciera.lib()
    return gpu_util


def _slice(host, dtype, shift):
    """A device copy of `host` at element `shift` of a guarded buffer."""
    buf = torch.full((host.size + 2 * GUARD,), 0x5A, dtype=dtype,
                     device="cuda")
    view = buf[shift:shift + host.size]
    view.copy_(torch.from_numpy(host.view(np.int16 if dtype == torch.int16
                                          else np.uint8)))
    return buf, view


def _guards_kept(buf, shift, size):
    b = buf.cpu().numpy()
    return (b[:shift] == 0x5A).all() and (b[shift + size:] == 0x5A).all()


@pytest.mark.parametrize("fp16", [False, True])
@pytest.mark.parametrize("B", [1, 16, 512, 4096])
@pytest.mark.parametrize("n,shift", [(3, 1), (2 * 16384 + 5, 3),
                                     (70_001, 7), (65_536, 5)])
def test_slices_at_odd_places(gu, orc, B, n, shift, fp16):
    from paper_2609_04609_amd import ciera, synth
    if fp16 and B == 1:
        pytest.skip("fp16 shards need B >= 16")
    R = 3
    if fp16:
        w = synth.normal_f16_bits(R * n, 0.02, n + B)
        w2 = synth.forced_bernoulli_f16_bits(w, 0.003, n + B + 1)
    else:
        w, w2 = gu.pair(R * n, n + B, c=0.003)
    wh, w2h = gu.host_u16(w), gu.host_u16(w2)
    split = orc.split_f16 if fp16 else orc.split
    enc_o = orc.encode_f16 if fp16 else orc.encode
    cache_h = split(wh)[0]
    flags = ciera.FP16 if fp16 else 0
    ws = ciera.Workspace(n, R, B)
    _, w2v = _slice(w2h, torch.int16, shift)
    shards = []
    for j in range(R):
        own = slice(j * n, (j + 1) * n)
        expect = enc_o(w2h[own], cache_h[own], B)
        for fused in (False, True):
            buf, c = _slice(cache_h[own], torch.uint8, shift + j)
            out = torch.full((int(ciera.ciera_encoded_bound(n, B, flags)),),
                             0xA5, dtype=torch.uint8, device="cuda")
            ciera.encode_t(w2v[own], c, B, ws, out, fp16=fp16,
                           update_cache=fused)
            got = gu.host_u8(out)
            np.testing.assert_array_equal(got[:expect.size], expect)
            assert (got[expect.size:] == 0xA5).all()
            assert _guards_kept(buf, shift + j, n)
            want = split(w2h[own])[0] if fused else cache_h[own]
            np.testing.assert_array_equal(gu.host_u8(c), want)
        # the cache update alone, from the bytes just encoded
        buf, c = _slice(cache_h[own], torch.uint8, shift + j)
        ciera.update_cache_t(c, out, n, B, ws, fp16=fp16)
        np.testing.assert_array_equal(gu.host_u8(c), split(w2h[own])[0])
        assert _guards_kept(buf, shift + j, n)
        # one shard of the three travels raw
        if j == 1:
            ciera.encode_t(w2v[own], None, B, ws, out, raw=True, fp16=fp16)
            expect = enc_o(w2h[own], None, B, raw=True)
            np.testing.assert_array_equal(gu.host_u8(out)[:expect.size],
                                          expect)
        shards.append(expect)
    g, offs = gu.gather(shards)
    offs = torch.from_numpy(offs.view(np.int64)).cuda()
    cbuf, cv = _slice(cache_h, torch.uint8, shift)
    obuf, ov = _slice(np.zeros(R * n, np.uint16), torch.int16, shift)
    ciera.decode_gathered_t(gu.dev_u8(g), offs, n, B, ov, cv, ws, fp16=fp16)
    np.testing.assert_array_equal(gu.host_u16(ov), w2h)
    np.testing.assert_array_equal(gu.host_u8(cv), split(w2h)[0])
    assert _guards_kept(cbuf, shift, R * n)
    assert _guards_kept(obuf, shift, R * n)
    assert ws.error() == 0
