"""The library's sources compiled as plain C++ against the host execution model
in ``tests/native/wave_host`` (fibers for threads, waves and workgroups in
ascending or descending order), with the C ABI on numpy buffers. Test
infrastructure: it shows what a kernel does in orders that the hardware may
choose, without a GPU."""
import ctypes
import os
import subprocess

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2609_04609_amd", "csrc")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"),
                     "lib/llvm/bin/clang++")
FLAGS = ["-x", "c++", "-std=c++17", "-O1", "-Wall", "-Werror",
         "-Wno-unused-function",
         "-I", os.path.join(HERE, "native", "wave_host"),
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]
LIB_SOURCES = [os.path.join(CSRC, f) for f in
               ("ciera_kernels.hip", "ciera_ans.hip", "ciera_api.cpp")]
ORDERS = [(w, g) for w in (0, 1) for g in (0, 1)]


def compile_lib(out, defines=()):
    """libciera as host code; `defines` as NAME=VALUE."""
    order = os.path.join(HERE, "native", "wave_host", "order.cpp")
    subprocess.run([CLANG, *FLAGS, *("-D" + d for d in defines), "-fPIC",
                    "-shared", *LIB_SOURCES, order, "-o", out], check=True)
    return out


def compile_exe(source, out):
    subprocess.run([CLANG, *FLAGS, source, "-o", out], check=True)
    return out


def buf(nbytes, fill=0):
    """A 64-byte aligned buffer of bytes."""
    b = np.full(nbytes + 64, fill, np.uint8)
    o = -b.ctypes.data % 64
    return b[o:o + nbytes]


class HostLib:
    """The calls the tests make, on numpy arrays (caches change in place)."""

    def __init__(self, path):
        from paper_2609_04609_amd import ciera
        self.c = ciera
        self.lib = ctypes.CDLL(path)
        for name, (res, args) in ciera._SIGS.items():
            if hasattr(self.lib, name):
                f = getattr(self.lib, name)
                f.restype, f.argtypes = res, args

    def order(self, waves_descend, groups_descend):
        self.lib.wave_host_order(waves_descend, groups_descend)

    def dispatched(self, call):
        """(launches, workgroups, the last kernel's address) of a call whose
        kernels are not run."""
        self.lib.wave_host_dry(1)
        call()
        last = self.lib.wave_host_last_kernel
        last.restype = ctypes.c_void_p
        seen = (self.lib.wave_host_launches(), self.lib.wave_host_groups(),
                last())
        self.lib.wave_host_dry(0)
        return seen

    def workspace(self, n, R, B, ans=False):
        return buf(self.lib.ciera_workspace_bytes(
            n, R, B, self.c.WS_ANS if ans else 0))

    @staticmethod
    def error(ws):
        return int(ws[:4].view(np.uint32)[0])

    def encode(self, w, cache, B, ws, flags=0):
        """(the output buffer, 0xA5 past the shard, and the shard's size)."""
        cap = self.lib.ciera_encoded_bound(w.size, B, flags & self.c.FP16)
        out, size = buf(cap, 0xA5), buf(8)
        rc = self.lib.ciera_encode(w.ctypes.data, cache.ctypes.data, w.size, B,
                                   flags, out.ctypes.data, cap,
                                   size.ctypes.data, ws.ctypes.data, ws.size,
                                   None)
        assert rc == 0, rc
        return out, int(size.view(np.uint64)[0])

    def encode_hashed(self, w, hashes, B, ws):
        cap = self.lib.ciera_encoded_bound(w.size, B, 0)
        out, size = buf(cap, 0xA5), buf(8)
        rc = self.lib.ciera_encode_hashed(
            w.ctypes.data, hashes.ctypes.data, hashes.ctypes.data, w.size, B,
            out.ctypes.data, cap, size.ctypes.data, ws.ctypes.data, ws.size,
            None)
        assert rc == 0, rc
        return out, int(size.view(np.uint64)[0])

    def ans_code(self, enc, n, B, ws):
        size = buf(8)
        rc = self.lib.ciera_ans_code(enc.ctypes.data, n, B, size.ctypes.data,
                                     ws.ctypes.data, ws.size, None)
        assert rc == 0, rc
        return int(size.view(np.uint64)[0])

    def decode(self, shards, n, B, cache, ws, flags=0):
        """The values of the shards (arrays of encoded bytes) back to back."""
        R = len(shards)
        gathered = buf(sum(s.size for s in shards))
        offs = np.cumsum([0] + [s.size for s in shards[:-1]]).astype(np.uint64)
        for o, s in zip(offs, shards):
            gathered[int(o):int(o) + s.size] = s
        out = np.zeros(R * n, np.uint16)
        rc = self.lib.ciera_decode_gathered(
            gathered.ctypes.data, gathered.size, offs.ctypes.data, R, n, B,
            flags, out.ctypes.data, cache.ctypes.data, ws.ctypes.data, ws.size,
            None)
        assert rc == 0, rc
        return out
