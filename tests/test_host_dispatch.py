"""Which kernels a call launches on both sides of the size lines, counted in the
host model without running them (tests/host_wave.py)."""
import pytest

from tests import host_wave as hw


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = hw.compile_lib(str(tmp_path_factory.mktemp("host") / "libciera.so"))
    return hw.HostLib(lib)


TILE = 16384


# one workgroup up to 49,152 values, in fp16 below B = 4096 up to 32,768
@pytest.mark.parametrize("kind,B,line", [
    ("exact", 1, 49_152), ("exact", 64, 49_152), ("exact", 4096, 49_152),
    ("hash", 16, 49_152), ("hash", 512, 49_152), ("fp16", 16, 32_768),
    ("fp16", 512, 32_768), ("fp16", 2048, 32_768), ("fp16", 4096, 49_152)])
def test_encode_in_one_launch(host, kind, B, line):
    c = host.c
    ws = host.workspace(line + 1, 1, B)
    out = hw.buf(host.lib.ciera_encoded_bound(
        line + 1, B, c.FP16 if kind == "fp16" else 0))
    p, o, w = hw.buf(64).ctypes.data, out.ctypes.data, ws.ctypes.data
    for n, launches in ((line, 1), (line + 1, 2)):
        def call():
            if kind == "hash":
                rc = host.lib.ciera_encode_hashed(p, p, p, n, B, o, out.size,
                                                  None, w, ws.size, None)
            else:
                rc = host.lib.ciera_encode(p, p, n, B,
                                           c.FP16 if kind == "fp16" else 0, o,
                                           out.size, None, w, ws.size, None)
            assert rc == 0
        assert host.dispatched(call)[0] == launches, n


# (kind, B, R, n, values a tile has): the merge of whole large tiles turns after
# 192 of them, what has a cut last tile, fp16 and the cache update after 255, B = 1
# at 16 MB of bitmap bytes counted in front of the tiles
@pytest.mark.parametrize("kind,B,R,n,tile", [
    ("bf16", 16, 16, 12 * TILE, 4096), ("bf16", 16, 16, 13 * TILE, TILE),
    ("bf16", 512, 192, TILE, 4096), ("bf16", 512, 193, TILE, TILE),
    ("bf16", 4096, 1, 192 * TILE, 4096), ("bf16", 4096, 1, 193 * TILE, TILE),
    ("bf16", 512, 16, 13 * TILE + 1, 4096),
    ("bf16", 512, 16, 15 * TILE - 4096, 4096),
    ("bf16", 512, 16, 16 * TILE - 1, TILE), ("bf16", 64, 255, 5, 4096),
    ("bf16", 64, 256, 4097, TILE),
    ("fp16", 512, 16, 15 * TILE, 4096), ("fp16", 512, 16, 16 * TILE, TILE),
    ("update", 512, 1, 255 * TILE, 4096), ("update", 512, 1, 256 * TILE, TILE),
    ("bf16", 1, 16, 15 * TILE, 4096), ("bf16", 1, 1, 64 * TILE, 4096),
    ("bf16", 1, 1, 65 * TILE, TILE)])
def test_decode_tiles(host, kind, B, R, n, tile):
    launches, groups, _ = host.dispatched(decode_call(host, kind, B, R, n))
    tiles = R * -(-n // tile)
    if B == 1 and tile == TILE:  # after the count kernel, four tiles a workgroup
        assert (launches, groups) == (2, tiles + R * -(-n // (4 * tile)))
    else:
        assert (launches, groups) == (1, tiles)


def decode_call(host, kind, B, R, n):
    flags = host.c.FP16 if kind == "fp16" else 0
    ws = host.workspace(n, R, B)
    one = hw.buf(64)  # nothing is read: no kernel runs
    p = one.ctypes.data

    def call():
        if kind == "update":
            rc = host.lib.ciera_update_cache(p, p, 64, n, B, 0, ws.ctypes.data,
                                             ws.size, None)
        else:
            rc = host.lib.ciera_decode_gathered(
                p, 64, p, R, n, B, flags, p, p, ws.ctypes.data, ws.size, None)
        assert rc == 0 and one is not None
    return call


@pytest.mark.parametrize("kind,B", [("bf16", 1), ("bf16", 16), ("bf16", 4096),
                                    ("fp16", 512)])
def test_one_small_tile_a_shard(host, kind, B):
    """Shards of up to 4096 values take the small tile's kernel at any number
    of shards, longer ones up to 255 large tiles."""
    def kernel(R, n):
        return host.dispatched(decode_call(host, kind, B, R, n))[2]
    small = kernel(1, 5)
    assert kernel(256, 5) == kernel(256, 4096) == kernel(65_535, 500) == small
    assert kernel(255, 4097) == small
    assert kernel(256, 4097) != small
