"""The kernels in every order of waves and workgroups: with waves in ascending
and descending order between barriers, and workgroups likewise, encodes,
decodes and rANS coding match the oracle byte for byte. What one order writes
over another's result is a missing barrier. Runs on the CPU (tests/host_wave.py);
no kernel here depends on the values' distribution, so small shards do."""
import os
import subprocess

import numpy as np
import pytest

from tests import host_wave as hw


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = hw.compile_lib(str(tmp_path_factory.mktemp("host") / "libciera.so"))
    return hw.HostLib(lib)


def _weights(n, seed):
    """Weights, and places whose exponents change."""
    rng = np.random.default_rng(seed)
    w = rng.integers(0, 1 << 16, n).astype(np.uint16)
    return w, rng.integers(0, n, 5)


def _stale(cache, at):
    """The cache as it was: other exponents at `at` and in the last block."""
    c = cache.copy()
    c[at] ^= 1
    if c.size:
        c[-1] ^= 1
    return c


def _before(w, at):
    """The weights of the iteration before: another exponent at `at`."""
    old = w.copy()
    old[at] ^= 1 << 7
    old[-1] ^= 1 << 7
    return old


# one workgroup up to 49,152 values, two kernels above; whole and short last
# blocks, chunks and octets
@pytest.mark.parametrize("n", [0, 1, 127, 4096, 4097, 20_001, 49_151, 49_152,
                               49_153, 70_000])
@pytest.mark.parametrize("B", [1, 16, 512, 1024, 4096])
def test_encode(host, orc, n, B):
    c = host.c
    w, at = _weights(max(n, 1), n + B)
    w = w[:n]
    ws = host.workspace(n, 1, B)
    cache = _stale(orc.split(w)[0], at if n else [])
    expect = orc.encode(w, cache, B)
    runs = [(0, w, cache, expect), (c.ENC_UPDATE_CACHE, w, cache, expect)]
    if B > 1:
        f = _stale(orc.split_f16(w)[0] & 0x1E, at if n else [])
        runs.append((c.FP16, w, f, orc.encode_f16(w, f, B)))
    for order in hw.ORDERS:
        host.order(*order)
        msg = f"n={n} B={B} order={order}"
        for flags, wf, cf, ex in runs:
            got, size = host.encode(wf, cf.copy(), B, ws, flags)
            assert size == ex.size, f"{msg} flags={flags}"
            np.testing.assert_array_equal(got[:size], ex, err_msg=msg)
            assert (got[size:] == 0xA5).all(), msg
        if B > 1 and n:
            h = orc.hash_blocks(_before(w, at), B).copy()
            old = h.copy()
            ex = orc.encode_hashed(w, old, B)[0]
            got, size = host.encode_hashed(w, h, B, ws)
            assert size == ex.size, msg
            np.testing.assert_array_equal(got[:size], ex, err_msg=msg)
        assert host.error(ws) == 0, msg


# small decode tiles (4096 values) and large ones, rANS below and above 16
# chunks, one shard of the gather raw
@pytest.mark.parametrize("n,R,B", [
    (4097, 3, 1), (4097, 3, 64), (4097, 3, 4096), (70_001, 2, 1),
    (70_001, 2, 64), (70_001, 2, 4096), (16_384, 256, 1), (16_384, 256, 512)])
def test_decode(host, orc, n, R, B):
    w, at = _weights(R * n, n + B)
    w2 = _before(w, at)
    cache = orc.split(w)[0]
    e2 = orc.split(w2)[0]
    own = [slice(j * n, (j + 1) * n) for j in range(R)]
    shards = [orc.encode(w2[s], None if j == 1 else cache[s], B, raw=j == 1)
              for j, s in enumerate(own)]
    ws = host.workspace(n, R, B)
    for order in hw.ORDERS if R < 8 else hw.ORDERS[:1]:
        host.order(*order)
        msg = f"n={n} R={R} B={B} order={order}"
        c = cache.copy()
        np.testing.assert_array_equal(host.decode(shards, n, B, c, ws), w2,
                                      err_msg=msg)
        np.testing.assert_array_equal(c, e2, err_msg=msg)
        assert host.error(ws) == 0, msg


@pytest.mark.parametrize("n", [5000, 65_536, 100_001])
def test_rans(host, orc, n):
    B = 512
    rng = np.random.default_rng(n)
    e = rng.choice([118, 119, 120, 121], n).astype(np.uint16)
    w = (e << 7) | rng.integers(0, 128, n).astype(np.uint16)
    cache = (e ^ 1).astype(np.uint8)  # every block changed
    plain = orc.encode(w, cache, B)
    expect = orc.ans_code(plain, n)
    ws = host.workspace(n, 2, B, ans=True)
    for order in hw.ORDERS:
        host.order(*order)
        msg = f"n={n} order={order}"
        enc = hw.buf(plain.size)
        enc[:] = plain
        size = host.ans_code(enc, n, B, ws)
        assert size == expect.size, msg
        np.testing.assert_array_equal(enc[:size], expect, err_msg=msg)
        c = np.concatenate([cache, cache])
        got = host.decode([enc[:size], enc[:size]], n, B, c, ws)
        np.testing.assert_array_equal(got, np.concatenate([w, w]), err_msg=msg)
        np.testing.assert_array_equal(c, np.concatenate([e, e]), err_msg=msg)
        assert host.error(ws) == 0, msg


def test_rans_size_decision_near_2_32(tmp_path):
    """A list of 2^32 - 256 bytes in K chunks: its streams are coded only if
    all of them together are shorter, also where their sum passes 2^32."""
    exe = hw.compile_exe(os.path.join(hw.HERE, "native", "ans_total.cpp"),
                         str(tmp_path / "ans_total"))
    n, K = (1 << 32) - 256, 1 << 20
    # 8 bits a symbol (2,048 words) and more; 1,919 make the streams 2^32 bytes,
    # 1,918 the whole section more than that, 1,916 less than the list
    words = [2048, 2100, 3136, 1920, 1919, 1918, 1916, 1000]
    r = subprocess.run([exe, *map(str, words)], capture_output=True, text=True,
                       check=True, timeout=300)
    rows = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    assert len(rows) == len(words)
    front = 64 + n + (1 << 20)  # header, values, bitmap (of n / 512 blocks)
    for w, (mode, total) in zip(words, rows):
        coded = 520 + 4 * K + K * ((256 + 2 * w + 3) // 4 * 4)
        if coded < n:
            assert (mode, total) == (2, front + (coded + 15) // 16 * 16), w
        else:
            assert (mode, total) == (0, front + n), w


def test_decode_of_builds_with_small_tiles(orc, tmp_path):
    """Built with 2 octets a lane, where large and small tiles are the same
    size, the decode at B = 1 still counts in front of its tiles."""
    host = hw.HostLib(hw.compile_lib(str(tmp_path / "libciera.so"),
                                     ["CIERA_DEC_OCT=2"]))
    for n, R in ((20_001, 2), (70_001, 20)):  # under and over 256 tiles
        w, at = _weights(R * n, n)
        w2 = _before(w, at)
        cache = orc.split(w)[0]
        shards = [orc.encode(w2[j * n:(j + 1) * n], cache[j * n:(j + 1) * n], 1)
                  for j in range(R)]
        ws = host.workspace(n, R, 1)
        ws[256:] = 0x5A  # what an earlier call may have left
        np.testing.assert_array_equal(host.decode(shards, n, 1, cache, ws), w2)
        np.testing.assert_array_equal(cache, orc.split(w2)[0])
        assert host.error(ws) == 0
